"""Outputs that share memory with inputs, single-queue lanes with the exchange by remote store, against the CPU oracle:
max-pool into the memory of its input, its backward into the memory of the gradient and the sign shares, element-wise
products and ReLU into memory that lies a few words beside an input.  Sizes of several workgroups."""
from ctypes import byref

import numpy as np
import pytest
import torch

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
    ln.set_exchange("put")
    yield ln
    ln.sync()
    ln.close()


def dev(mpc, shares):
    return tuple(mpc.to_device(s) for s in shares)


def buffers(words, parties):
    return [torch.zeros(words, dtype=torch.int64, device="cuda:0") for _ in range(parties)]


def place(mpc, bufs, at, shares):
    """The shares at word `at` of the buffers (views)."""
    views = tuple(b[at:at + s.size] for b, s in zip(bufs, shares))
    for v, s in zip(views, shares):
        v.copy_(mpc.to_device(np.ascontiguousarray(s).reshape(-1)))
    torch.cuda.synchronize()
    return views


def equal(mpc, got, want):
    for i, w in enumerate(want):
        g = mpc.to_host(got[i].clone()).reshape(w.shape)
        assert np.array_equal(g, w), f"party {i} differs at {np.argwhere(g != w)[:3].tolist()} of {w.size}"


def kit(parties):
    if parties == 2:
        return synth.share_additive, synth.deal_relu_material, "material_to_device", "_material", "_share", "pack_material"
    return synth.share_additive3, synth.deal_relu3_material, "material_to_device", "_material3", "_share3", "pack_material3"


def triple(rng, n, share):
    A, B = synth.rand_words(rng, n), synth.rand_words(rng, n)
    return share(rng, A), share(rng, B), share(rng, A * B)


@pytest.mark.parametrize("parties", [2, 3])
@pytest.mark.parametrize("packed", [False, True])
@pytest.mark.parametrize("at", [0, 70])
def test_maxpool_into_its_input(mpc, lane, at, packed, parties):
    B, H, W, C = 2, 16, 24, 33
    n = B * (H // 2) * (W // 2) * C
    print(f"maxpool into its input at {at}, packed={packed}, {parties} parties", flush=True)
    rng = np.random.default_rng(at + parties)
    share, deal, to_dev, marshal, sh, pack = kit(parties)
    xs = share(rng, synth.normal_fixed(rng, (B, H, W, C), 4.0))
    m1, m2 = deal(rng, 2 * n), deal(rng, n)
    want = (oracle.maxpool2x2 if parties == 2 else oracle.maxpool2x2_3)(xs, m1, m2)
    d1, d2 = getattr(mpc, to_dev)(m1), getattr(mpc, to_dev)(m2)
    if packed:
        d1, d2 = getattr(lane, pack)(d1), getattr(lane, pack)(d2)
    bufs = buffers(4 * n, parties)
    x = place(mpc, bufs, 0, xs)
    y = tuple(b[at:at + n] for b in bufs)
    L, s = mpc.lib(), "_msb" if packed else ""
    ma, mb = getattr(mpc, marshal)(d1, 2 * n, packed), getattr(mpc, marshal)(d2, n, packed)
    share_of = getattr(mpc, sh)
    if parties == 2:
        lane.reserve(getattr(L, "mpc_maxpool" + s + "_workspace_bytes")(B, H, W, C))
        rc = getattr(L, "mpc_maxpool2x2" + s)(lane._h, share_of(x), byref(ma), byref(mb), share_of(y), B, H, W, C, 0)
    else:
        lane.reserve(getattr(L, "mpc_maxpool3" + s + "_workspace_bytes")(B, H, W, C))
        rc = getattr(L, "mpc_maxpool3" + s)(lane._h, share_of(x), byref(ma), byref(mb), share_of(y), B, H, W, C)
    lane._check(rc)
    lane.sync()
    equal(mpc, y, want)


@pytest.mark.parametrize("parties", [2, 3])
@pytest.mark.parametrize("where", ["gradient", "signs1", "signs2", "triple"])
def test_maxpool_backward_into_an_operand(mpc, lane, where, parties):
    shape = B, H, W, C = 2, 16, 24, 33
    n = B * (H // 2) * (W // 2) * C
    print(f"maxpool backward into {where}, {parties} parties", flush=True)
    rng = np.random.default_rng(n + parties)
    share, _, _, _, sh, _ = kit(parties)
    signs = lambda k: share(rng, rng.integers(0, 2, size=k).astype(np.uint64))
    g, s1, s2 = share(rng, synth.normal_fixed(rng, (B, H // 2, W // 2, C), 0.5)), signs(2 * n), signs(n)
    t1, t2 = triple(rng, 2 * n, share), triple(rng, n, share)
    want = (oracle.maxpool2x2_backward if parties == 2 else oracle.maxpool2x2_backward3)(g, s1, s2, t1, t2, shape)
    args = [dev(mpc, v) for v in (g, s1, s2, *t1, *t2)]
    k = {"gradient": 0, "signs1": 1, "signs2": 2, "triple": 4}[where]
    bufs = buffers(4 * n + 64, parties)
    args[k] = place(mpc, bufs, 64 if k else 0, (g, s1, s2, *t1, *t2)[k])
    gx = tuple(b[:4 * n] for b in bufs)
    L, c = mpc.lib(), getattr(mpc, sh)
    lane.reserve((L.mpc_maxpool_backward_workspace_bytes if parties == 2 else L.mpc_maxpool3_backward_workspace_bytes)(*shape))
    call = L.mpc_maxpool2x2_backward if parties == 2 else L.mpc_maxpool3_backward
    lane._check(call(lane._h, *(c(v) for v in args), c(gx), *shape))
    lane.sync()
    equal(mpc, gx, want)


@pytest.mark.parametrize("parties", [2, 3])
@pytest.mark.parametrize("shift", [-129, -1, 64, 1000])
def test_mul_beside_an_operand(mpc, lane, shift, parties):
    n = 9000
    print(f"mul shifted by {shift}, {parties} parties", flush=True)
    rng = np.random.default_rng(n + shift)
    share, _, _, _, sh, _ = kit(parties)
    x, y = (share(rng, synth.normal_fixed(rng, n, 2.0)) for _ in range(2))
    t = triple(rng, n, share)
    want = (oracle.beaver_mul if parties == 2 else oracle.beaver_mul3)(x, y, *t)
    bufs = buffers(n + 2000, parties)
    xd = place(mpc, bufs, 1000, x)
    z = tuple(b[1000 + shift:1000 + shift + n] for b in bufs)
    args = dev(mpc, y), *(dev(mpc, v) for v in t)
    (lane.mul if parties == 2 else lane.mul3)(xd, *args, out=z)
    lane.sync()
    equal(mpc, z, want)


@pytest.mark.parametrize("parties", [2, 3])
@pytest.mark.parametrize("packed", [False, True])
@pytest.mark.parametrize("where,shift", [("x", 130), ("x", -1), ("r", 65), ("own array", 0)])
def test_relu_beside_an_operand(mpc, lane, where, shift, packed, parties):
    """own array: the output is exactly an input's array, which stays one launch."""
    n = 9000
    print(f"relu output beside {where} by {shift}, packed={packed}, {parties} parties", flush=True)
    rng = np.random.default_rng(n + shift)
    share, deal, to_dev, _, _, pack = kit(parties)
    xs = share(rng, synth.normal_fixed(rng, n, 4.0))
    mat = deal(rng, n)
    want = (oracle.relu if parties == 2 else oracle.relu3)(xs, mat).y
    md = getattr(mpc, to_dev)(mat)
    if packed:
        md = getattr(lane, pack)(md)
    bufs = buffers(n + 400, parties)
    x = dev(mpc, xs)
    key = {"x": None, "r": "r" if parties == 2 else "r1", "own array": "ma"}[where]
    if key is None:
        x = place(mpc, bufs, 200, xs)
    else:
        md[key] = place(mpc, bufs, 200, mat[key])
    y = tuple(b[200 + shift:200 + shift + n] for b in bufs)
    (lane.relu if parties == 2 else lane.relu3)(x, md, out=y, packed=packed)
    lane.sync()
    equal(mpc, y, want)
