"""Products with at most 32 output rows run on a tile of 32 x 128: the edges of that tile, contractions with fewer steps
than the ring has slots, split ones, and convolutions whose output has few pixels, against the oracle bit for bit."""
import numpy as np
import pytest

from helpers import deal_conv, deal_matmul, oracle_conv, oracle_matmul

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mpc():
    from paper_2209_13643_amd import mpc as m
    return m


@pytest.fixture(scope="module")
def lane(mpc):
    ln = mpc.Lane(0, single_queue=True)
    ln.set_exchange("put")
    yield ln
    ln.sync()
    ln.close()


def dev(mpc, pair):
    return (mpc.to_device(pair[0]), mpc.to_device(pair[1]))


def same(mpc, lane, got, want, what):
    lane.sync()
    for i in range(2):
        g = mpc.to_host(got[i]).reshape(want[i].shape)
        assert np.array_equal(g, want[i]), f"{what}: party {i} differs in {(g != want[i]).sum()} of {g.size} words"


@pytest.mark.parametrize("M,K,N,batch", [
    (1, 1, 1, None), (1, 16, 128, None), (2, 33, 129, None), (31, 64, 127, None), (32, 96, 128, None), (32, 97, 257, None),
    (33, 96, 128, None), (2, 4096, 300, None), (17, 1500, 640, 3), (32, 32, 32, 96), (5, 64, 513, 7),
])
def test_matmul(mpc, lane, M, K, N, batch):
    rng = np.random.default_rng(M * 1000003 + K * 1009 + N)
    d = deal_matmul(rng, M, K, N, batch=batch)
    args = [dev(mpc, d[k]) for k in ("x", "y", "a", "b", "c")]
    for flags, bits in ((0, 0), (mpc.MPC_TRUNCATE, 16)):
        z = lane.beaver_matmul(*args, flags=flags)
        same(mpc, lane, z, oracle_matmul(d, bits), f"{M}x{K}x{N} batch {batch} flags {flags}")


@pytest.mark.parametrize("M,K,N,batch", [
    (8, 64, 64, 512), (8, 64, 64, 511), (32, 40, 33, 600), (33, 40, 33, 600), (3, 128, 65, 300), (4, 129, 64, 513), (1, 1, 1, 512),
])
def test_batched_products_of_few_rows(mpc, lane, M, K, N, batch):
    """Around the rule that gives batched products of at most 64 columns and short contractions the 64 x 64 tile."""
    rng = np.random.default_rng(M + K + N + batch)
    d = deal_matmul(rng, M, K, N, batch=batch)
    x, y, a, b, c = (dev(mpc, d[k]) for k in ("x", "y", "a", "b", "c"))
    same(mpc, lane, lane.beaver_matmul(x, y, a, b, c), oracle_matmul(d), f"{batch} x {M}x{K}x{N}")
    right, left = lane.prepare_matmul(a, b, None)
    z = lane.beaver_matmul_folded(x, y, a, b, (lane.fold_matmul(a, b, c), c[1]), right, left)
    same(mpc, lane, z, oracle_matmul(d), f"folded, {batch} x {M}x{K}x{N}")


@pytest.mark.parametrize("B,H,W,Cin,Cout,k,pad,stride", [
    (1, 2, 2, 40, 130, 3, 1, 1), (8, 2, 2, 17, 128, 3, 1, 1), (1, 8, 8, 5, 64, 3, 1, 2), (2, 7, 7, 64, 70, 1, 0, 2), (1, 5, 6, 3, 200, 3, 1, 1),
])
def test_conv(mpc, lane, B, H, W, Cin, Cout, k, pad, stride):
    rng = np.random.default_rng(B * 7919 + H * 31 + Cin + Cout)
    d = deal_conv(rng, B, H, W, Cin, Cout, k, k, pad, stride)
    args = [dev(mpc, d[n]) for n in ("x", "y", "a", "b", "c")]
    z = lane.conv2d(*args, pad=pad, stride=stride, flags=mpc.MPC_TRUNCATE)
    same(mpc, lane, z, oracle_conv(d, 16), f"conv {B}x{H}x{W}x{Cin}->{Cout} k{k} s{stride}")
