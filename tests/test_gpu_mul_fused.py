"""GPU parity of the element-wise products as one launch (single-queue lanes, exchange by remote store) against the CPU
oracle at the edges of their tiles: fewer elements than a wave, ragged last tiles, the change from one to two elements
per thread (131 072 | 131 073), an output that overwrites an input; and the max-pool backward built on them."""
import numpy as np
import pytest

import oracle
from paper_2209_13643_amd import synth

pytestmark = pytest.mark.gpu
SIZES = [1, 2, 63, 64, 65, 4097, 131072, 131073, 262144 + 129]


@pytest.fixture(scope="module")
def mpc():
    from paper_2209_13643_amd import mpc as m
    return m


@pytest.fixture()
def lane(mpc):
    ln = mpc.Lane(0, single_queue=True)
    ln.set_exchange("put")
    yield ln
    ln.sync()
    ln.close()


def dev(mpc, shares):
    return tuple(mpc.to_device(s) for s in shares)


def equal(mpc, got, want):
    for i, w in enumerate(want):
        g = mpc.to_host(got[i]).reshape(w.shape)
        assert np.array_equal(g, w), f"party {i} differs at {np.argwhere(g != w)[:3].tolist()} of {w.size}"


def triple(rng, n, share):
    A, B = synth.rand_words(rng, n), synth.rand_words(rng, n)
    return share(rng, A), share(rng, B), share(rng, A * B)


def sign_shares(rng, n, share):
    return share(rng, rng.integers(0, 2, size=n).astype(np.uint64))


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("truncate", [False, True])
def test_one_launch_mul(mpc, lane, n, truncate):
    print(f"mul n={n} truncate={truncate}", flush=True)
    rng = np.random.default_rng(n)
    x, y = (synth.share_additive(rng, synth.normal_fixed(rng, n, 2.0)) for _ in range(2))
    t = triple(rng, n, synth.share_additive)
    want = oracle.beaver_mul(x, y, *t)
    if truncate:
        want = oracle.truncate(want, 16)
    xd = dev(mpc, x)
    z = lane.mul(xd, dev(mpc, y), *(dev(mpc, v) for v in t), flags=mpc.MPC_TRUNCATE if truncate else 0, out=xd if n % 2 else None)
    lane.sync()
    equal(mpc, z, want)


@pytest.mark.parametrize("parties", [2, 3])
@pytest.mark.parametrize("n", SIZES)
def test_one_launch_relu_backward(mpc, lane, n, parties):
    print(f"relu backward n={n} parties={parties}", flush=True)
    rng = np.random.default_rng(n)
    share = synth.share_additive if parties == 2 else synth.share_additive3
    g, s, t = share(rng, synth.normal_fixed(rng, n, 0.5)), sign_shares(rng, n, share), triple(rng, n, share)
    want = (oracle.relu_backward if parties == 2 else oracle.relu_backward3)(g, s, *t)
    run = lane.relu_backward if parties == 2 else lane.relu3_backward
    gx = run(dev(mpc, g), dev(mpc, s), *(dev(mpc, v) for v in t))
    lane.sync()
    equal(mpc, gx, want)


@pytest.mark.parametrize("n", [1, 64, 65, 131073])
def test_one_launch_mul_three_parties(mpc, lane, n):
    print(f"mul3 n={n}", flush=True)
    rng = np.random.default_rng(n)
    x, y = (synth.share_additive3(rng, synth.normal_fixed(rng, n, 2.0)) for _ in range(2))
    t = triple(rng, n, synth.share_additive3)
    z = lane.mul3(dev(mpc, x), dev(mpc, y), *(dev(mpc, v) for v in t))
    lane.sync()
    equal(mpc, z, oracle.beaver_mul3(x, y, *t))


@pytest.mark.parametrize("parties", [2, 3])
@pytest.mark.parametrize("shape", [(1, 2, 2, 1), (1, 2, 2, 64), (1, 2, 2, 65), (2, 4, 6, 5), (3, 16, 16, 33), (9, 32, 32, 64)])
def test_one_launch_maxpool_backward(mpc, lane, shape, parties):
    print(f"maxpool backward {shape} parties={parties}", flush=True)
    B, H, W, C = shape
    n = B * (H // 2) * (W // 2) * C
    rng = np.random.default_rng(n)
    share = synth.share_additive if parties == 2 else synth.share_additive3
    g = share(rng, synth.normal_fixed(rng, (B, H // 2, W // 2, C), 0.5))
    s1, s2 = sign_shares(rng, 2 * n, share), sign_shares(rng, n, share)
    t1, t2 = triple(rng, 2 * n, share), triple(rng, n, share)
    want = (oracle.maxpool2x2_backward if parties == 2 else oracle.maxpool2x2_backward3)(g, s1, s2, t1, t2, shape)
    run = lane.maxpool2x2_backward if parties == 2 else lane.maxpool3_backward
    gx = run(dev(mpc, g), dev(mpc, s1), dev(mpc, s2), tuple(dev(mpc, v) for v in t1), tuple(dev(mpc, v) for v in t2), shape)
    lane.sync()
    equal(mpc, gx, want)
