"""Which form a two-party product's GEMM launch takes, on the CPU: the built library's host side on a stand-in for the HIP
runtime.  Products and convolutions with few tiles and long contractions that measured faster on the larger tiles take
them, others the form in which the waves of a workgroup share a tile's contraction; split over workgroups, that form never
gives an XCD more workgroups than it has compute units."""
import pytest

import fake_hip

CALLS = r'''
flags = 1
lib.mpc_matmul_workspace_bytes.restype = lib.mpc_conv2d_workspace_bytes.restype = c_size_t
lib.mpc_matmul_workspace_bytes.argtypes = [c_int] * 4
lib.mpc_conv2d_workspace_bytes.argtypes = [c_int] * 9
lib.mpc_beaver_matmul_prepared.argtypes = [c_void_p] + [Share] * 4 + [c_void_p] * 2 + [c_int] * 6
lib.mpc_conv2d_prepared.argtypes = [c_void_p] + [Share] * 4 + [c_void_p] * 2 + [c_int] * 11
assert lib.mpc_ctx_set_exchange(ctx, 1) == 0
big = array(1 << 38)
share = lambda: Share((c_void_p * 2)(big, big + (1 << 37)))

def product(M, K, N, batch=1, flags=1):
    ws = lib.mpc_matmul_workspace_bytes(M, K, N, batch)
    assert lib.mpc_ctx_set_workspace(ctx, array(ws), ws) == 0
    assert lib.mpc_beaver_matmul_prepared(ctx, share(), share(), share(), share(), big, big, M, K, N, batch, 1, flags) == 0
    return [n for n in launches() if "gemm" in n]

def convolution(B, HW, Cin, Cout, k, stride):
    g = (B, HW, HW, Cin, Cout, k, k, k // 2, stride)
    ws = lib.mpc_conv2d_workspace_bytes(*g)
    assert lib.mpc_ctx_set_workspace(ctx, array(ws), ws) == 0
    assert lib.mpc_conv2d_prepared(ctx, share(), share(), share(), share(), big, big, *g, 1, 1) == 0
    return [n for n in launches() if "gemm" in n]
'''
FOLDED = 1 | 16


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    d = tmp_path_factory.mktemp("fake")
    return lambda body: fake_hip.run(d, CALLS + body)


def sliced(names):
    assert len(names) == 1, names
    return "k_sliced_gemm" in names[0]


def test_long_contractions_on_the_larger_tiles(run):
    """The launch, us, larger tiles / shared: 64 x 8000 x 2000 125 / 155, 1073 x 12347 x 89 188 / 232, 316 x 25053 x 158
    204 / 226, 119 x 16989 x 800 208 / 277, the strided convolution 60 / 80."""
    r = run('''
for s in ((64, 8000, 2000), (1073, 12347, 89), (316, 25053, 158), (119, 16989, 800)):
    result[str(s)] = product(*s)
result["conv"] = convolution(34, 6, 368, 276, 3, 2)
''')
    for what, names in r.items():
        assert not sliced(names), (what, names)


def test_few_rows_and_few_steps(run):
    """More than 512 tiles of 32 x 32 of both parties and at most 6 steps: the 32 x 128 tiles, unless they need a second round
    or are half empty."""
    tiles = ((8, 8, 240, 57), (1, 21, 595, 21), (12, 66, 111, 102))
    shared = ((8, 8, 240, 30), (8, 150, 240, 57), (8, 8, 64, 200), (8, 8, 129, 100), (40, 8, 240, 30), (33, 8, 140, 50))
    r = run(f'''
for s in {tiles + shared}:
    result[str(s)] = product(*s)
''')
    for s in tiles:
        assert not sliced(r[str(s)]), s
    for s in shared:
        assert sliced(r[str(s)]), (s, r[str(s)])


def test_long_contractions_shared(run):
    r = run('''
for s in ((2, 25088, 10), (64, 2048, 128), (60, 8000, 400), (44, 17839, 164), (72, 3891, 1231)):
    result[str(s)] = product(*s)
result["conv"] = convolution(4, 7, 256, 256, 3, 1)
''')
    for what, names in r.items():
        assert sliced(names), (what, names)


def test_one_round_of_workgroups(run):
    """Every party's workgroups are dealt to the eight XCDs of 32 compute units in eights."""
    r = run(f'''
for s in ((22, 21586, 472), (28, 10597, 559), (2, 4097, 708), (6, 12597, 539), (3, 5457, 529), (44, 17839, 164), (30, 1100, 4000)):
    result[str(s)] = product(*s, flags={FOLDED})
''')
    split = 0
    for what, names in r.items():
        if sliced(names):
            split += 1
            assert int(names[0].split("@")[1]) <= 256, (what, names)
    assert split >= 3
