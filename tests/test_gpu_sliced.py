"""GEMM launches with few output tiles: the waves of a workgroup share one 32 x 32 tile's contraction.  Edges of the tile,
fewer steps than waves, the two numbers of waves (256 | 257 tiles of both parties), the longest contraction it takes (64 K
steps) without a choice by cost, contractions split over workgroups as well, taps that cross k blocks, one, two and three parties, partial sums of a two-phase call; each
shape also on the tiles of larger products, which the tuning call leaves as the only ones.  Against the oracle bit for bit."""
import numpy as np
import pytest

import oracle
from helpers import deal_conv, deal_matmul, oracle_conv, oracle_matmul
from paper_2209_13643_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mpc():
    from paper_2209_13643_amd import mpc as m
    return m


@pytest.fixture(params=["few tiles", "large tiles"])
def lane(mpc, request):
    ln = mpc.Lane(0, single_queue=True)
    ln.set_exchange("put")
    if request.param == "large tiles":
        mpc.set_gemm_small_tile(0, 512)
    yield ln
    mpc.set_gemm_small_tile()
    ln.sync()
    ln.close()


def dev(mpc, pair):
    return tuple(mpc.to_device(p) for p in pair)


def same(mpc, lane, got, want, what):
    lane.sync()
    for i in range(len(want)):
        g = mpc.to_host(got[i]).reshape(want[i].shape)
        assert np.array_equal(g, want[i]), f"{what}: party {i} differs in {(g != want[i]).sum()} of {g.size} words"


@pytest.mark.parametrize("M,K,N,batch", [
    (1, 1, 1, None), (31, 17, 33, None), (32, 64, 32, None), (33, 128, 31, None), (64, 250, 70, None), (65, 512, 129, None),
    (40, 1008, 20, None), (40, 1024, 33, None), (40, 1025, 20, None), (500, 40, 256, None), (513, 40, 256, None), (40, 48, 36, 32),
    (2, 300, 100, 3), (5, 4100, 33, None), (65, 2500, 40, None), (20, 1300, 24, 3), (2, 12000, 130, None), (100, 1100, 1000, None), (70, 100, 500, 3),
    (300, 100, 70, 3),
])
def test_products(mpc, lane, M, K, N, batch):
    print(f"sliced {M}x{K}x{N} batch {batch}", flush=True)
    d = deal_matmul(np.random.default_rng(M * 1000003 + K * 1009 + N), M, K, N, batch=batch)
    x, y, a, b, c = (dev(mpc, d[k]) for k in ("x", "y", "a", "b", "c"))
    same(mpc, lane, lane.beaver_matmul(x, y, a, b, c), oracle_matmul(d), "plain")
    same(mpc, lane, lane.beaver_matmul(x, y, a, b, c, flags=0), oracle_matmul(d, 0), "plain, no truncation")
    right, left = lane.prepare_matmul(a, b, None)
    cf = (lane.fold_matmul(a, b, c), c[1])
    same(mpc, lane, lane.beaver_matmul_folded(x, y, a, b, cf, right, left), oracle_matmul(d), "folded")
    f = lane.open(lane.sub(y, b))
    z = lane.beaver_matmul(x, None, a, b, c, f_public=f, flags=mpc.MPC_TRUNCATE | mpc.MPC_TWO_PHASE)
    same(mpc, lane, z, oracle_matmul(d), "two phases")


@pytest.mark.parametrize("B,H,W,Cin,Cout,k,pad,stride", [
    (1, 4, 4, 3, 20, 3, 1, 1), (2, 5, 7, 17, 33, 3, 1, 1), (1, 9, 9, 40, 64, 3, 0, 2), (2, 6, 6, 33, 40, 1, 0, 2), (3, 4, 4, 48, 96, 3, 1, 1),
    (1, 6, 5, 16, 32, 5, 2, 1), (8, 12, 12, 20, 130, 3, 1, 1), (2, 4, 4, 200, 40, 3, 1, 1), (1, 5, 5, 500, 33, 3, 1, 2),
    (3, 1, 1, 17, 1, 5, 2, 2), (1, 1, 5, 40, 33, 3, 1, 1), (1, 1, 1, 33, 20, 3, 1, 1), (2, 1, 1, 20, 70, 7, 3, 1), (1, 2, 1, 5, 9, 7, 3, 1), (1, 3, 2, 18, 40, 7, 3, 2),
])
def test_convolutions(mpc, lane, B, H, W, Cin, Cout, k, pad, stride):
    print(f"sliced conv {B}x{H}x{W}x{Cin}->{Cout} k{k} s{stride}", flush=True)
    d = deal_conv(np.random.default_rng(B * 7919 + H * 31 + Cin + Cout), B, H, W, Cin, Cout, k, k, pad, stride)
    x, w, a, b, c = (dev(mpc, d[n]) for n in ("x", "y", "a", "b", "c"))
    same(mpc, lane, lane.conv2d(x, w, a, b, c, pad, stride), oracle_conv(d, 16), "plain")
    right, left = lane.prepare_conv2d(a, b, lane.open(lane.sub(w, b)), pad, stride)
    cf = (lane.fold_conv2d(a, b, c, pad, stride), c[1])
    z = lane.conv2d_prepared(x, a, cf, right, left, k, k, pad, stride, flags=mpc.MPC_TRUNCATE | mpc.MPC_FOLDED)
    same(mpc, lane, z, oracle_conv(d, 16), "folded")


@pytest.mark.parametrize("M,K,N", [(1, 5, 3), (70, 200, 40), (33, 1024, 65), (20, 5000, 50)])
def test_one_and_three_parties(mpc, lane, M, K, N):
    rng = np.random.default_rng(M + K)
    L, R = synth.rand_words(rng, (M, K)), synth.rand_words(rng, (K, N))
    got = lane.ring_matmul(mpc.to_device(L), mpc.to_device(R))
    lane.sync()
    assert np.array_equal(mpc.to_host(got), oracle.ring_matmul(L, R))
    x, y, a, b = (synth.rand_words(rng, s) for s in ((M, K), (K, N), (M, K), (K, N)))
    sh = {k: synth.share_additive3(rng, v) for k, v in (("x", x), ("y", y), ("a", a), ("b", b), ("c", oracle.ring_matmul(a, b)))}
    z = lane.beaver_matmul3(*(dev(mpc, sh[k]) for k in ("x", "y", "a", "b", "c")))
    same(mpc, lane, z, oracle.beaver_matmul3(*(sh[k] for k in ("x", "y", "a", "b", "c"))), "three parties")
