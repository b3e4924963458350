"""GPU parity of the secure ReLU as one launch (single-queue lanes, exchange by remote store) against the CPU oracle at
the sizes where its tiling can go wrong: fewer elements than a wave, ragged last tiles, the change from one to two
elements per thread (65 536 | 65 537), several tiles per workgroup, and an output that overwrites the input."""
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
    ln.set_exchange("put")
    yield ln
    ln.sync()
    ln.close()


def dev(mpc, pair):
    return tuple(mpc.to_device(p) for p in pair)


def equal(mpc, got, want, what):
    for i, w in enumerate(want):
        g = mpc.to_host(got[i]).reshape(w.shape)
        assert np.array_equal(g, w), f"{what}: party {i} differs at {np.argwhere(g != w)[:3].tolist()} of {w.size}"


SIZES = [1, 2, 3, 63, 64, 65, 127, 65535, 65536, 65537, 131072, 131073, 262144 + 130]


@pytest.mark.parametrize("adder", ["kogge-stone", "tree"])
@pytest.mark.parametrize("n", SIZES)
def test_one_launch_relu(mpc, lane, n, adder):
    print(f"one-launch relu n={n} {adder}", flush=True)
    rng = np.random.default_rng(n)
    xs = synth.share_additive(rng, synth.normal_fixed(rng, n, 4.0))
    mat = synth.deal_relu_material(rng, n)
    want = oracle.relu(xs, mat, adder=adder)
    lane.set_adder(adder)
    x = dev(mpc, xs)
    y, sb, sa = lane.relu(x, mpc.material_to_device(mat), want_sign=True, out=x if n % 2 else None)
    lane.sync()
    equal(mpc, y, want.y, "output")
    equal(mpc, sb, want.s_bit, "sign bit share")
    equal(mpc, sa, want.s_arith, "sign arithmetic share")


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 255, 4097, 65536, 65537, 65536 + 256 + 65, 131072, 131073, 131072 + 128 + 65, 524288 + 3])
def test_one_launch_sign_only_relu(mpc, lane, n):
    """The packed chain changes from one to four elements per lane at 65 536 | 65 537; beyond it the last n mod 256
    elements run one per lane."""
    print(f"one-launch sign-only relu n={n}", flush=True)
    rng = np.random.default_rng(n)
    xs = synth.share_additive(rng, synth.normal_fixed(rng, n, 4.0))
    mat = synth.deal_relu_material(rng, n)
    want = oracle.relu(xs, mat)
    x = dev(mpc, xs)
    y, sb, sa = lane.relu(x, lane.pack_material(mpc.material_to_device(mat)), want_sign=True, packed=True, out=x if n % 2 else None)
    lane.sync()
    equal(mpc, y, want.y, "output")
    equal(mpc, sb, want.s_bit, "sign bit share")
    equal(mpc, sa, want.s_arith, "sign arithmetic share")


@pytest.mark.parametrize("packed", [False, True])
@pytest.mark.parametrize("n", [1, 2, 63, 65, 32768, 32769, 65536 + 129, 98304, 98305, 98304 + 193])
def test_one_launch_relu_three_parties(mpc, lane, n, packed):
    """Three parties: one to two elements per lane at 32 768 | 32 769 (whole words) and 98 304 | 98 305 (packed)."""
    print(f"one-launch three-party relu n={n} packed={packed}", flush=True)
    rng = np.random.default_rng(n)
    xs = synth.share_additive3(rng, synth.normal_fixed(rng, n, 4.0))
    mat = synth.deal_relu3_material(rng, n)
    want = oracle.relu3(xs, mat)
    md = mpc.material_to_device(mat)
    x = dev(mpc, xs)
    y, sb, sa = lane.relu3(x, lane.pack_material3(md) if packed else md, want_sign=True, packed=packed, out=x if n % 2 else None)
    lane.sync()
    equal(mpc, y, want.y, "output")
    equal(mpc, sb, want.s_bit, "sign bit share")
    equal(mpc, sa, want.s_arith, "sign arithmetic share")


@pytest.mark.parametrize("parties,chain", [(2, "kogge-stone"), (2, "tree"), (2, "packed"), (3, "kogge-stone"), (3, "packed")])
@pytest.mark.parametrize("shape", [(1, 2, 2, 1), (1, 2, 2, 63), (1, 2, 2, 64), (1, 2, 2, 65), (2, 4, 6, 5), (3, 6, 4, 11), (2, 16, 16, 33),
                                   (5, 32, 32, 64)])
def test_one_launch_maxpool(mpc, lane, shape, parties, chain):
    """64 outputs per wave: ragged last tiles (also of the packed words), channel counts around a wave, several tiles per
    workgroup; outputs and both levels' sign shares."""
    print(f"one-launch maxpool {shape} {chain} parties={parties}", flush=True)
    B, H, W, C = shape
    n_out = B * (H // 2) * (W // 2) * C
    rng = np.random.default_rng(n_out)
    X = synth.normal_fixed(rng, shape, 4.0)
    if parties == 2:
        xs, m1, m2 = synth.share_additive(rng, X), synth.deal_relu_material(rng, 2 * n_out), synth.deal_relu_material(rng, n_out)
        want, s1, s2 = oracle.maxpool2x2(xs, m1, m2, want_signs=True, adder="tree" if chain == "tree" else "kogge-stone")
        lane.set_adder("tree" if chain == "tree" else "kogge-stone")
        pool, pack = lane.maxpool2x2, lane.pack_material
    else:
        xs, m1, m2 = synth.share_additive3(rng, X), synth.deal_relu3_material(rng, 2 * n_out), synth.deal_relu3_material(rng, n_out)
        want, s1, s2 = oracle.maxpool2x2_3(xs, m1, m2, want_signs=True)
        pool, pack = lane.maxpool3, lane.pack_material3
    d1, d2 = mpc.material_to_device(m1), mpc.material_to_device(m2)
    if chain == "packed":
        d1, d2 = pack(d1), pack(d2)
    y, g1, g2 = pool(dev(mpc, xs), d1, d2, packed=chain == "packed", want_signs=True)
    lane.sync()
    equal(mpc, y, want, "output")
    equal(mpc, g1, s1, "first level's sign shares")
    equal(mpc, g2, s2, "second level's sign shares")


@pytest.mark.parametrize("chain", ["kogge-stone", "tree", "packed"])
@pytest.mark.parametrize("queues", ["one", "three"])
@pytest.mark.parametrize("n", [1, 33, 63, 64, 65, 100, 4097, 65536, 65537, 131072 + 129, 262144, 262145])
def test_copies_inside_the_launch(mpc, n, queues, chain):
    """Exchange by copies, the default: up to 2^18 elements the rounds and their copies are one launch, beyond it launches of
    their own.  On a workspace of exactly the queried size between guard areas."""
    from ctypes import c_void_p
    import torch
    print(f"copying relu n={n} {queues} {chain}", flush=True)
    rng = np.random.default_rng(n)
    xs = synth.share_additive(rng, synth.normal_fixed(rng, n, 4.0))
    mat = synth.deal_relu_material(rng, n)
    want = oracle.relu(xs, mat, adder="tree" if chain == "tree" else "kogge-stone")
    packed = chain == "packed"
    ln = mpc.Lane(0, single_queue=queues == "one")
    ln.set_adder("tree" if chain == "tree" else "kogge-stone")
    md = mpc.material_to_device(mat)
    if packed:
        md = ln.pack_material(md)
    nbytes = (mpc.lib().mpc_relu_msb_workspace_bytes if packed else mpc.lib().mpc_relu_workspace_bytes)(n)
    if n <= 1 << 18:         # room for the one launch: four buffers a workgroup, four rows of its lanes' words (packed: two of whole words)
        per_lane = 1 if n <= 65536 else 4 if packed else 2
        tiles = n // 256 + (n % 256 + 63) // 64 if packed and per_lane == 4 else (n + 64 * per_lane - 1) // (64 * per_lane)
        assert nbytes >= min(tiles, 1024) * 4 * (2 if packed else 4) * 64 * per_lane * 8
    guard = 4096
    buf = torch.full((nbytes + 2 * guard + 256,), 0xA5, dtype=torch.uint8, device="cuda:0")
    at = guard + (-(buf.data_ptr() + guard)) % 256
    ln.sync()
    torch.cuda.synchronize()
    ln._check(mpc.lib().mpc_ctx_set_workspace(ln._h, c_void_p(buf.data_ptr() + at), nbytes))
    ln._ws, ln._ws_bytes = buf, nbytes
    x = dev(mpc, xs)
    torch.cuda.synchronize()
    y, sb, sa = ln.relu(x, md, want_sign=True, packed=packed, out=x if n % 2 else None)
    ln.sync()
    equal(mpc, y, want.y, "output")
    equal(mpc, sb, want.s_bit, "sign bit share")
    equal(mpc, sa, want.s_arith, "sign arithmetic share")
    b = buf.cpu().numpy()
    assert (b[:at] == 0xA5).all() and (b[at + nbytes:] == 0xA5).all(), "written outside the workspace"
    ln.close()


@pytest.mark.parametrize("exchange", ["put", "copy"])
@pytest.mark.parametrize("n", [65536, 65537, 65536 + 255, 65536 + 256 + 65, 262144 - 1, 262144 + 191, 600000])
def test_sign_only_relu_four_elements_per_lane(mpc, n, exchange):
    """The packed chain takes four elements per lane from 65 537 elements on, its last n mod 256 one per lane; several tiles
    per workgroup from 262 145 on."""
    print(f"sign-only relu n={n} {exchange}", flush=True)
    rng = np.random.default_rng(n)
    xs = synth.share_additive(rng, synth.normal_fixed(rng, n, 4.0))
    mat = synth.deal_relu_material(rng, n)
    want = oracle.relu(xs, mat)
    ln = mpc.Lane(0, single_queue=True)
    ln.set_exchange(exchange)
    x = dev(mpc, xs)
    y, sb, sa = ln.relu(x, ln.pack_material(mpc.material_to_device(mat)), want_sign=True, packed=True, out=x if n % 2 else None)
    ln.sync()
    equal(mpc, y, want.y, "output")
    equal(mpc, sb, want.s_bit, "sign bit share")
    equal(mpc, sa, want.s_arith, "sign arithmetic share")
    ln.close()
