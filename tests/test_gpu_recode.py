"""GPU parity of the digit-plane recoders at the edges of their tiles (64 rows, four 16-wide k blocks, filter taps),
through the plain ring products that read such planes."""
import numpy as np
import pytest

import oracle
from paper_2209_13643_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mpc():
    from paper_2209_13643_amd import mpc as m
    return m


@pytest.fixture()
def lane(mpc):
    ln = mpc.Lane(0, single_queue=True)
    yield ln
    ln.sync()
    ln.close()


@pytest.mark.parametrize("Cin,Cout", [(1, 16), (3, 17), (64, 32), (65, 33), (70, 63), (5, 64), (66, 65), (64, 200)])
@pytest.mark.parametrize("k", [1, 3])
def test_filter_with_swapped_channel_roles(mpc, lane, Cin, Cout, k):
    """The input gradient reads the forward filter with k = Cout contiguous: the tile recoder runs per filter tap once
    a tap has two k blocks (Cout > 16), with ragged rows (Cin), ragged k and the padding block behind the last tap."""
    print(f"grad_x planes Cin={Cin} Cout={Cout} k={k}", flush=True)
    rng = np.random.default_rng(100 * Cin + Cout)
    g = synth.rand_words(rng, (2, 5, 6, Cout)); w = synth.rand_words(rng, (k, k, Cin, Cout))
    want = oracle.ring_conv2d_grad_x(g, w, (2, 5, 6, Cin), k // 2, 1)
    got = lane.ring_conv2d_grad_x(mpc.to_device(g), mpc.to_device(w), (2, 5, 6, Cin), k // 2, 1)
    lane.sync()
    assert np.array_equal(mpc.to_host(got), want)


@pytest.mark.parametrize("M,K,N", [(1, 1, 1), (3, 15, 5), (63, 16, 65), (64, 17, 64), (65, 63, 1), (70, 65, 129), (130, 130, 3)])
def test_ragged_units(mpc, lane, M, K, N):
    """Rows, k blocks and columns one short of, at and one past a tile, in both recoders."""
    print(f"ragged units {M}x{K}x{N}", flush=True)
    rng = np.random.default_rng(M + K + N)
    L = synth.rand_words(rng, (M, K)); R = synth.rand_words(rng, (K, N))
    got = lane.ring_matmul(mpc.to_device(L), mpc.to_device(R))
    lane.sync()
    assert np.array_equal(mpc.to_host(got), oracle.ring_matmul(L, R))


@pytest.mark.parametrize("hw,stride,pad", [(4, 1, 1), (5, 2, 0), (7, 1, 0), (6, 2, 1)])
def test_transposed_im2col(mpc, lane, hw, stride, pad):
    """Filter gradient: 16 output pixels per unit cross image rows, images and the end of the batch."""
    print(f"im2col_t hw={hw} stride={stride} pad={pad}", flush=True)
    rng = np.random.default_rng(hw + stride)
    ho = (hw + 2 * pad - 3) // stride + 1
    x = synth.rand_words(rng, (3, hw, hw, 5)); g = synth.rand_words(rng, (3, ho, ho, 7))
    got = lane.ring_conv2d_grad_w(mpc.to_device(x), mpc.to_device(g), 3, 3, pad, stride)
    lane.sync()
    assert np.array_equal(mpc.to_host(got), oracle.ring_conv2d_grad_w(x, g, 3, 3, pad, stride))


@pytest.mark.parametrize("M,K,N", [(1, 1, 5), (2, 3, 4), (65, 4, 7), (63, 62, 33), (64, 64, 16), (66, 68, 20), (130, 129, 9), (300, 200, 31)])
@pytest.mark.parametrize("call", ["folded", "plain", "activations"])
def test_masked_recodings_of_ragged_tiles(mpc, call, M, K, N):
    """Exchange by remote store: the recodings that mask, send and open on the way, with threads past the last k, word-wise
    and 16-byte accesses and rows past the last one."""
    from helpers import deal_matmul, oracle_matmul
    print(f"masked recoding {call} {M}x{K}x{N}", flush=True)
    lane = mpc.Lane(0, single_queue=True)
    lane.set_exchange("put")
    d = deal_matmul(np.random.default_rng(M + K + N), M, K, N)
    want = oracle_matmul(d)
    x, y, a, b, c = (tuple(mpc.to_device(p) for p in d[k]) for k in ("x", "y", "a", "b", "c"))
    if call == "plain":
        z = lane.beaver_matmul(x, y, a, b, c)
    else:
        f = lane.open(lane.sub(y, b)) if call == "folded" else None
        right, left = lane.prepare_matmul(a, b, f)
        cf = (lane.fold_matmul(a, b, c), c[1])
        if call == "folded":
            z = lane.beaver_matmul_prepared(x, a, cf, right, left, flags=mpc.MPC_TRUNCATE | mpc.MPC_FOLDED)
        else:
            z = lane.beaver_matmul_folded(x, y, a, b, cf, right, left)
    lane.sync()
    for i in range(2):
        assert np.array_equal(mpc.to_host(z[i]), want[i]), f"party {i}"
    lane.close()


@pytest.mark.parametrize("B,H,W,Cin", [(1, 1, 1, 3), (2, 2, 2, 5), (1, 3, 5, 64), (3, 4, 4, 65), (2, 16, 16, 7), (1, 5, 17, 33), (2, 31, 3, 20), (1, 32, 32, 3)])
def test_transposed_im2col_of_three_by_three_filters(mpc, lane, B, H, W, Cin):
    """Filter gradient of a 3x3 filter with stride 1 and padding 1: units of 16 pixels that cross image rows and images,
    neighbours outside the row, the end of the batch, images narrower and wider than a unit."""
    print(f"im2col3_t {B}x{H}x{W}x{Cin}", flush=True)
    rng = np.random.default_rng(B * H * W + Cin)
    x = synth.rand_words(rng, (B, H, W, Cin)); g = synth.rand_words(rng, (B, H, W, 6))
    got = lane.ring_conv2d_grad_w(mpc.to_device(x), mpc.to_device(g), 3, 3, 1, 1)
    lane.sync()
    assert np.array_equal(mpc.to_host(got), oracle.ring_conv2d_grad_w(x, g, 3, 3, 1, 1))
