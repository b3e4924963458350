"""Ordering on a lane with three streams: calls without tiles run on stream 0, tiled calls on all three, and both kinds
follow each other on the same buffers; a caller that holds party 1's stream sees party 1's output on it."""
import numpy as np
import pytest
import torch

import oracle
from helpers import deal_matmul, oracle_matmul
from paper_2209_13643_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mpc():
    from paper_2209_13643_amd import mpc as m
    return m


def dev(mpc, pair):
    return tuple(mpc.to_device(p) for p in pair)


@pytest.mark.parametrize("handles", [False, True])
@pytest.mark.parametrize("chunks", [(1, 3), (3, 1), (1, 1), (3, 3)])
def test_tiled_and_untiled_calls_in_turn(mpc, chunks, handles):
    """Linear layer then ReLU with and without tiles, several rounds over the same output buffers."""
    print(f"tiles {chunks} handles={handles}", flush=True)
    rng = np.random.default_rng(7)
    M, K, N = 96, 200, 160
    lane = mpc.Lane(0)
    s1 = torch.cuda.ExternalStream(lane.stream(1)) if handles else None
    d = deal_matmul(rng, M, K, N)
    mat = synth.deal_relu_material(rng, M * N)
    want_z = oracle_matmul(d); want = oracle.relu(want_z, mat).y
    args = [dev(mpc, d[k]) for k in ("x", "y", "a", "b", "c")]
    md = mpc.material_to_device(mat)
    z = tuple(torch.empty((M, N), dtype=torch.int64, device="cuda:0") for _ in range(2))
    y = tuple(torch.empty_like(z[0]) for _ in range(2))
    torch.cuda.synchronize()
    for _ in range(5):
        lane.beaver_matmul(*args, n_chunks=chunks[0], out=z)
        lane.relu(z, md, n_chunks=chunks[1], out=y)
    if handles:
        s1.synchronize()
        assert np.array_equal(mpc.to_host(y[1]).reshape(-1), want[1].reshape(-1)), "party 1's stream alone"
    lane.sync()
    for i in range(2):
        assert np.array_equal(mpc.to_host(z[i]), want_z[i]) and np.array_equal(mpc.to_host(y[i]).reshape(-1), want[i].reshape(-1)), i
    lane.close()


def long_relu(mpc, lane, n=1 << 20):
    """An untiled call of about a millisecond: (material kept alive, output, expected shares)."""
    rng = np.random.default_rng(11)
    xs = synth.share_additive(rng, synth.normal_fixed(rng, n, 4.0))
    mat = synth.deal_relu_material(rng, n)
    x, md = dev(mpc, xs), mpc.material_to_device(mat)
    y = tuple(torch.zeros(n, dtype=torch.int64, device="cuda:0") for _ in range(2))
    lane.relu(x, md, out=y); lane.sync()                 # kernels loaded, workspace in place
    for t in y:
        t.zero_()
    torch.cuda.synchronize()
    lane.relu(x, md, out=y)
    return (x, md), y, oracle.relu(xs, mat).y


@pytest.mark.parametrize("which", [1, 2])
def test_stream_handle_taken_after_the_call(mpc, which):
    """The handle of another stream, asked for after an untiled call, is ordered behind that call's outputs."""
    print(f"stream {which} taken after the call", flush=True)
    lane = mpc.Lane(0)
    keep, y, want = long_relu(mpc, lane)
    s = torch.cuda.ExternalStream(lane.stream(which))
    with torch.cuda.stream(s):
        got = [t.clone() for t in y]
    s.synchronize()
    for i in range(2):
        assert np.array_equal(mpc.to_host(got[i]), want[i]), i
    lane.sync()
    lane.close()


@pytest.mark.parametrize("which", [1, 2])
def test_stream_replaced_after_the_call(mpc, which):
    """A caller's stream put in the place of the lane's own one starts behind what the lane has issued."""
    print(f"stream {which} replaced after the call", flush=True)
    lane = mpc.Lane(0)
    keep, y, want = long_relu(mpc, lane)
    s = torch.cuda.Stream()
    handles = [None, None, None]
    handles[which] = s.cuda_stream
    lane._check(mpc.lib().mpc_ctx_set_streams(lane._h, *handles))
    with torch.cuda.stream(s):
        got = [t.clone() for t in y]
    s.synchronize()
    for i in range(2):
        assert np.array_equal(mpc.to_host(got[i]), want[i]), i
    lane.sync()
    lane.close()


@pytest.mark.parametrize("which", [0, 1, 2])
def test_wait_torch_covers_streams_the_caller_holds(mpc, which):
    print(f"wait_torch, stream {which}", flush=True)
    lane = mpc.Lane(0)
    s = torch.cuda.ExternalStream(lane.stream(which))
    x = torch.zeros(1 << 26, dtype=torch.int64, device="cuda:0")
    torch.cuda.synchronize()
    for _ in range(20):
        x += 1                                           # some milliseconds on torch's stream
    lane.wait_torch()
    with torch.cuda.stream(s):
        got = x[-1000:].clone()
    s.synchronize()
    assert (got == 20).all()
    torch.cuda.synchronize()
    lane.close()
