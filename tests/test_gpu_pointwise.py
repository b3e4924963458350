"""1x1 convolutions of stride 1 without padding and with an even number of channel blocks run as plain products; odd
numbers of blocks, strides and paddings keep the gather.  Both sides of that line, against the oracle bit for bit."""
import numpy as np
import pytest

from helpers import deal_conv, oracle_conv

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


@pytest.mark.parametrize("B,H,W,Cin,Cout,pad,stride", [
    (1, 5, 7, 17, 40, 0, 1), (2, 9, 5, 32, 65, 0, 1), (3, 13, 11, 64, 129, 0, 1), (1, 30, 31, 100, 256, 0, 1),     # plain
    (2, 9, 5, 48, 65, 0, 1), (1, 5, 7, 16, 40, 0, 1), (2, 9, 9, 32, 65, 0, 2), (2, 7, 7, 32, 65, 1, 1),            # gather
])
def test_pointwise_conv(mpc, lane, B, H, W, Cin, Cout, pad, stride):
    rng = np.random.default_rng(B * 7919 + H * 31 + Cin + Cout)
    d = deal_conv(rng, B, H, W, Cin, Cout, 1, 1, pad, stride)
    x, w, a, b, c = (dev(mpc, d[n]) for n in ("x", "y", "a", "b", "c"))
    z = lane.conv2d(x, w, a, b, c, pad, stride)
    same(mpc, lane, z, oracle_conv(d), f"1x1 conv {B}x{H}x{W}x{Cin}->{Cout} pad {pad} stride {stride}")
    f_public = mpc.to_device((d["y"][0] - d["b"][0]) + (d["y"][1] - d["b"][1]))
    right, left = lane.prepare_conv2d(a, b, f_public, pad, stride)
    z = lane.conv2d_prepared(x, a, c, right, left, 1, 1, pad, stride)
    same(mpc, lane, z, oracle_conv(d), "prepared")
