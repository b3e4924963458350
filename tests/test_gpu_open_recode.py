"""The one launch that masks, exchanges and recodes the opened operands of a call (single-queue lanes, exchange by remote
store), folded or plain, against the oracle bit for bit: its tiles are 128 rows x 16 k, 64 x 32 and 32 x 64 by the width of the operand,
128 rows x 16 k for operands stored [K][N]; few rows, ragged edges, the zero row of a convolution's planes at the start of a
tile of its own, several tiles per workgroup, words at odd addresses."""
import numpy as np
import pytest
import torch

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


def odd(mpc, array):
    """The words at an address that is 8 but not 16 bytes aligned."""
    t = mpc.to_device(array)
    buf = torch.empty(t.numel() + 2, dtype=t.dtype, device=t.device)
    out = buf[1:1 + t.numel()].view(t.shape)
    if out.data_ptr() % 16 == 0:
        out = buf[2:2 + t.numel()].view(t.shape)
    out.copy_(t)
    torch.cuda.synchronize()
    return out


def dev(mpc, pair, at=None):
    return tuple((at or mpc.to_device)(*((mpc, p) if at else (p,))) for p in pair)


def same(mpc, lane, got, want, what):
    lane.sync()
    for i in range(2):
        g = mpc.to_host(got[i]).reshape(want[i].shape)
        assert np.array_equal(g, want[i]), f"{what}: party {i} differs in {(g != want[i]).sum()} of {g.size} words"


@pytest.mark.parametrize("M,K,N,batch", [
    (16, 65, 40, None), (17, 64, 33, None), (31, 66, 129, None), (32, 128, 16, None), (33, 130, 128, None), (49, 63, 20, None),
    (64, 32, 65, None), (65, 17, 63, None), (129, 33, 5, None), (128, 16, 64, None), (130, 15, 50, None), (300, 3, 200, None),
    (2, 2000, 30, None), (20, 70, 24, 5), (3, 200, 129, 4), (24640, 64, 1, None), (5, 7, 1500, 3),
    (3, 9000, 4, None), (17, 3000, 8, 5), (3, 13000, 7, None),
])
def test_products(mpc, lane, M, K, N, batch):
    """Both operands opened by the call, and the left one alone; folded, and plain with the masks' planes."""
    print(f"one-launch opening {M}x{K}x{N} batch {batch}", flush=True)
    d = deal_matmul(np.random.default_rng(M * 1000003 + K * 1009 + N), M, K, N, batch=batch)
    want = oracle_matmul(d)
    at = odd if K % 2 else None
    x, y, a, b = (dev(mpc, d[k], at) for k in ("x", "y", "a", "b"))
    c = dev(mpc, d["c"])
    cf = (lane.fold_matmul(a, b, c), c[1])
    right, left = lane.prepare_matmul(a, b, None)
    same(mpc, lane, lane.beaver_matmul_folded(x, y, a, b, cf, right, left), want, "both operands")
    right, left = lane.prepare_matmul(a, b, lane.open(lane.sub(y, b)))
    z = lane.beaver_matmul_prepared(x, a, cf, right, left, flags=mpc.MPC_TRUNCATE | mpc.MPC_FOLDED)
    same(mpc, lane, z, want, "left operand")
    same(mpc, lane, lane.beaver_matmul(x, y, a, b, c), want, "plain")
    z = lane.beaver_matmul(x, None, a, b, c, f_public=lane.open(lane.sub(y, b)))
    same(mpc, lane, z, want, "plain, weight mask opened ahead")


@pytest.mark.parametrize("trans", ["x", "y", "both"])
def test_transposed_operands(mpc, lane, trans):
    """Either operand with its rows or its k contiguous."""
    M, K, N = 70, 45, 150
    d = deal_matmul(np.random.default_rng(5), M, K, N, batch=2)
    tr = lambda pair: tuple(np.ascontiguousarray(p.transpose(0, 2, 1)) for p in pair)
    fx, fy = trans in ("x", "both"), trans in ("y", "both")
    x, a = (dev(mpc, tr(d[k]) if fx else d[k]) for k in ("x", "a"))
    y, b = (dev(mpc, tr(d[k]) if fy else d[k]) for k in ("y", "b"))
    c = dev(mpc, d["c"])
    flags = (mpc.MPC_TRANS_X if fx else 0) | (mpc.MPC_TRANS_Y if fy else 0)
    right, left = lane.prepare_matmul(a, b, None, flags=flags)
    cf = (lane.fold_matmul(a, b, c, flags=flags), c[1])
    z = lane.beaver_matmul_folded(x, y, a, b, cf, right, left, flags=flags | mpc.MPC_TRUNCATE)
    same(mpc, lane, z, oracle_matmul(d), f"transposed {trans}")
    z = lane.beaver_matmul(x, y, a, b, c, flags=flags | mpc.MPC_TRUNCATE)
    same(mpc, lane, z, oracle_matmul(d), f"transposed {trans}, plain")


@pytest.mark.parametrize("B,H,W,Cin,Cout,k", [
    (2, 8, 8, 3, 20, 3), (1, 16, 8, 16, 33, 3), (2, 8, 8, 17, 16, 1), (1, 8, 8, 32, 16, 3), (2, 4, 4, 40, 24, 3), (3, 5, 7, 65, 10, 1),
])
def test_convolutions(mpc, lane, B, H, W, Cin, Cout, k):
    print(f"one-launch opening conv {B}x{H}x{W}x{Cin}", flush=True)
    d = deal_conv(np.random.default_rng(B * H * W + Cin), B, H, W, Cin, Cout, k, k, k // 2, 1)
    x, w, a, b, c = (dev(mpc, d[n]) for n in ("x", "y", "a", "b", "c"))
    right, left = lane.prepare_conv2d(a, b, lane.open(lane.sub(w, b)), k // 2, 1)
    cf = (lane.fold_conv2d(a, b, c, k // 2, 1), c[1])
    z = lane.conv2d_prepared(x, a, cf, right, left, k, k, k // 2, 1, flags=mpc.MPC_TRUNCATE | mpc.MPC_FOLDED)
    same(mpc, lane, z, oracle_conv(d, 16), "conv")
    same(mpc, lane, lane.conv2d(x, w, a, b, c, k // 2, 1), oracle_conv(d, 16), "conv, plain")      # opens the filter too


@pytest.mark.parametrize("M,K,N", [(1, 700, 40), (17, 64, 33), (33, 130, 128), (65, 17, 63), (129, 33, 70), (300, 3, 200), (64, 1300, 40), (1000, 300, 5), (70000, 1, 3), (3, 40000, 4)])
def test_three_parties(mpc, lane, M, K, N):
    """Masks' planes of all parties (plain), the opened words alone (prepared), the weight mask opened ahead."""
    import oracle
    from paper_2209_13643_amd import synth
    print(f"one-launch opening, three parties {M}x{K}x{N}", flush=True)
    rng = np.random.default_rng(M * 31 + K)
    A, Bm = synth.rand_words(rng, (M, K)), synth.rand_words(rng, (K, N))
    words = dict(x=synth.rand_words(rng, (M, K)), y=synth.rand_words(rng, (K, N)), a=A, b=Bm, c=oracle.ring_matmul(A, Bm))
    sh = {k: synth.share_additive3(rng, v) for k, v in words.items()}
    want = oracle.beaver_matmul3(*(sh[k] for k in ("x", "y", "a", "b", "c")))
    x, y, a, b, c = (tuple(mpc.to_device(p) for p in sh[k]) for k in ("x", "y", "a", "b", "c"))

    def check(z, what):
        lane.sync()
        for i in range(3):
            g = mpc.to_host(z[i])
            assert np.array_equal(g, want[i]), f"{what}: party {i} differs in {(g != want[i]).sum()} of {g.size} words"

    check(lane.beaver_matmul3(x, y, a, b, c), "plain")
    f = lane.open3(lane.sub3(y, b))
    check(lane.beaver_matmul3(x, y, a, b, c, f_public=f), "weight mask opened ahead")
    right, left = lane.prepare_matmul3(a, b, f)
    check(lane.beaver_matmul3_prepared(x, a, c, right, left), "prepared")


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 130, 131072, 131073, 131072 + 129, 262144 + 77, 600001])
def test_three_party_rescale(mpc, lane, n):
    """One launch: fewer elements than a wave, ragged tiles, one or two elements per thread, several tiles per workgroup."""
    import oracle
    from paper_2209_13643_amd import synth
    print(f"one-launch rescale n={n}", flush=True)
    rng = np.random.default_rng(n)
    z = synth.share_additive3(rng, synth.normal_fixed(rng, n, 300.0) * np.uint64(1 << 16))
    r, rt = synth.deal_trunc3_pair(rng, n)
    want = oracle.truncate3(z, r, rt)
    up = lambda t: tuple(mpc.to_device(p) for p in t)
    got = lane.truncate3(up(z), up(r), up(rt))
    lane.sync()
    for i in range(3):
        assert np.array_equal(mpc.to_host(got[i]), want[i]), f"party {i}"
