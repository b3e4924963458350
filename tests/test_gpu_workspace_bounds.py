"""Calls on a workspace that is a part of a larger buffer, of exactly the size the query names: nothing is written outside
it and the results are the oracle's.  Single-queue lanes, exchange by remote store, sizes around one wave."""
from ctypes import c_void_p

import numpy as np
import pytest
import torch

import oracle
from paper_2209_13643_amd import synth

pytestmark = pytest.mark.gpu
GUARD, FILL = 8192, 0xA5


@pytest.fixture(scope="module")
def mpc():
    from paper_2209_13643_amd import mpc as m
    return m


class Guarded:
    """A single-queue lane whose workspace of `nbytes` lies between two guard areas."""

    def __init__(self, mpc, nbytes, exchange="put"):
        self.lane = mpc.Lane(0, single_queue=True)
        self.lane.set_exchange(exchange)
        self.buf = torch.full((nbytes + 2 * GUARD + 256,), FILL, dtype=torch.uint8, device="cuda:0")
        self.at = GUARD + (-(self.buf.data_ptr() + GUARD)) % 256
        torch.cuda.synchronize()
        self.lane._check(mpc.lib().mpc_ctx_set_workspace(self.lane._h, c_void_p(self.buf.data_ptr() + self.at), nbytes))
        self.nbytes = nbytes

    def check(self):
        self.lane.sync()
        b = self.buf.cpu().numpy()
        assert (b[:self.at] == FILL).all(), "written before the workspace"
        behind = b[self.at + self.nbytes:]
        assert (behind == FILL).all(), f"written behind the workspace, up to byte {int(np.flatnonzero(behind != FILL)[-1])}"
        self.lane.close()


def dev(mpc, shares):
    return tuple(mpc.to_device(s) for s in shares)


def empty(shape, parties):
    return tuple(torch.empty(shape, dtype=torch.int64, device="cuda:0") for _ in range(parties))


def equal(mpc, got, want):
    for i, w in enumerate(want):
        assert np.array_equal(mpc.to_host(got[i]).reshape(w.shape), w), f"party {i}"


def triple(rng, n, share):
    A, B = synth.rand_words(rng, n), synth.rand_words(rng, n)
    return share(rng, A), share(rng, B), share(rng, A * B)


@pytest.mark.parametrize("parties", [2, 3])
@pytest.mark.parametrize("n", [1, 16, 17, 64, 65])
def test_maxpool_backward_stays_inside_its_workspace(mpc, n, parties):
    print(f"maxpool backward, {n} outputs, {parties} parties", flush=True)
    shape, L = (1, 2, 2, n), mpc.lib()
    rng = np.random.default_rng(n)
    share = synth.share_additive if parties == 2 else synth.share_additive3
    signs = lambda k: share(rng, rng.integers(0, 2, size=k).astype(np.uint64))
    g, s1, s2 = share(rng, synth.normal_fixed(rng, (1, 1, 1, n), 0.5)), signs(2 * n), signs(n)
    t1, t2 = triple(rng, 2 * n, share), triple(rng, n, share)
    want = (oracle.maxpool2x2_backward if parties == 2 else oracle.maxpool2x2_backward3)(g, s1, s2, t1, t2, shape)
    query, call, c = ((L.mpc_maxpool_backward_workspace_bytes, L.mpc_maxpool2x2_backward, mpc._share) if parties == 2 else
                      (L.mpc_maxpool3_backward_workspace_bytes, L.mpc_maxpool3_backward, mpc._share3))
    args = [dev(mpc, v) for v in (g, s1, s2, *t1, *t2)]
    gx = empty(shape, parties)
    w = Guarded(mpc, query(*shape))
    w.lane._check(call(w.lane._h, *(c(v) for v in args), c(gx), *shape))
    w.check()
    equal(mpc, gx, want)


def up(v):
    return (v + 255) // 256 * 256


def mul3(n):
    return 18 * up(8 * n)


def relu3(n):
    return 3 * (6 * up(8 * n) + 3 * up(32 * n) + 4 * up(n)) + 6 * up(32 * n)


# bytes of the arrays of the launch sequences: enough for every call, whatever the receive buffers of one launch need
ARRAYS = {
    "mul3": mul3,
    "relu3": relu3,
    "maxpool": lambda n: 2 * (2 * up(16 * n) + 2 * up(8 * n)) + 2 * (2 * up(64 * n) + 3 * up(2 * n) + 2 * up(16 * n)) + 2 * up(64 * n),
    "maxpool3": lambda n: 3 * (2 * up(16 * n) + 2 * up(8 * n)) + relu3(2 * n),
    "maxpool_backward": lambda n: 2 * (up(8 * n) + 2 * up(16 * n)) + 8 * up(16 * n),
    "maxpool3_backward": lambda n: 3 * (up(8 * n) + 2 * up(16 * n)) + mul3(2 * n),
}


@pytest.mark.parametrize("exchange", ["copy", "put"])
@pytest.mark.parametrize("n", [1, 8, 9, 32, 33])
@pytest.mark.parametrize("call", sorted(ARRAYS))
def test_workspace_of_the_arrays_alone(mpc, call, n, exchange):
    print(f"{call} n={n} {exchange}", flush=True)
    from ctypes import byref
    L, rng = mpc.lib(), np.random.default_rng(n)
    three = "3" in call
    share, c = (synth.share_additive3, mpc._share3) if three else (synth.share_additive, mpc._share)
    deal, marshal = (synth.deal_relu3_material, mpc._material3) if three else (synth.deal_relu_material, mpc._material)
    parties, shape = 3 if three else 2, (1, 2, 2, n)
    w = Guarded(mpc, ARRAYS[call](n), exchange)
    h = w.lane._h
    signs = lambda k: share(rng, rng.integers(0, 2, size=k).astype(np.uint64))
    if call == "mul3":
        x, y, t = share(rng, synth.rand_words(rng, n)), share(rng, synth.rand_words(rng, n)), triple(rng, n, share)
        args, out, want = [dev(mpc, v) for v in (x, y, *t)], empty(n, 3), oracle.beaver_mul3(x, y, *t)
        rc = L.mpc_mul3(h, *(c(v) for v in args), c(out), n)
    elif call == "relu3":
        x, mat = share(rng, synth.normal_fixed(rng, n, 4.0)), deal(rng, n)
        args, out, want = (dev(mpc, x), mpc.material_to_device(mat)), empty(n, 3), oracle.relu3(x, mat).y
        rc = L.mpc_relu3(h, c(args[0]), byref(marshal(args[1], n)), c(out), n, None, None)
    elif call in ("maxpool", "maxpool3"):
        x, m1, m2 = share(rng, synth.normal_fixed(rng, shape, 4.0)), deal(rng, 2 * n), deal(rng, n)
        args, out = (dev(mpc, x), mpc.material_to_device(m1), mpc.material_to_device(m2)), empty((1, 1, 1, n), parties)
        want = (oracle.maxpool2x2_3 if three else oracle.maxpool2x2)(x, m1, m2)
        ms = byref(marshal(args[1], 2 * n)), byref(marshal(args[2], n))
        rc = L.mpc_maxpool3(h, c(args[0]), *ms, c(out), *shape) if three else L.mpc_maxpool2x2(h, c(args[0]), *ms, c(out), *shape, 0)
    else:
        g, s1, s2 = share(rng, synth.normal_fixed(rng, (1, 1, 1, n), 0.5)), signs(2 * n), signs(n)
        t1, t2 = triple(rng, 2 * n, share), triple(rng, n, share)
        args, out = [dev(mpc, v) for v in (g, s1, s2, *t1, *t2)], empty(shape, parties)
        want = (oracle.maxpool2x2_backward3 if three else oracle.maxpool2x2_backward)(g, s1, s2, t1, t2, shape)
        rc = (L.mpc_maxpool3_backward if three else L.mpc_maxpool2x2_backward)(h, *(c(v) for v in args), c(out), *shape)
    assert rc == 0, f"refused with {rc}"
    w.check()
    equal(mpc, out, want)
