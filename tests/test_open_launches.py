"""The launches that open and recode a linear layer's operands under the exchange by remote store, on the CPU: the built
library's host side on a stand-in for the HIP runtime."""
import pytest

import fake_hip

CALLS = r'''
for q in ("mpc_matmul_workspace_bytes", "mpc_matmul3_workspace_bytes"):
    getattr(lib, q).restype = c_size_t; getattr(lib, q).argtypes = [c_int] * 4
lib.mpc_beaver_matmul.argtypes = [c_void_p] + [Share] * 6 + [c_int] * 4 + [c_void_p, c_int, c_int]
lib.mpc_beaver_matmul3.argtypes = [c_void_p] + [Share3] * 6 + [c_int] * 4 + [c_void_p, c_int]
lib.mpc_conv2d_grad_x_workspace_bytes.restype = c_size_t; lib.mpc_conv2d_grad_x_workspace_bytes.argtypes = [c_int] * 9
lib.mpc_conv2d_grad_x.argtypes = [c_void_p] + [Share] * 6 + [c_int] * 9 + [c_void_p, c_int, c_int]
assert lib.mpc_ctx_set_exchange(ctx, 1) == 0
big = array(1 << 38)
share = lambda: Share((c_void_p * 2)(big, big + (1 << 37)))
share3 = lambda: Share3((c_void_p * 3)(big, big + (1 << 36), big + (1 << 37)))

def query(parties, *s):
    return (lib.mpc_matmul_workspace_bytes if parties == 2 else lib.mpc_matmul3_workspace_bytes)(*s)

def product(parties, ws, *s, f_public=None):
    """rc, launches, workgroups of the opening launch (0: none)"""
    assert lib.mpc_ctx_set_workspace(ctx, array(ws), ws) == 0
    if parties == 2: rc = lib.mpc_beaver_matmul(ctx, *[share() for _ in range(6)], *s, f_public, 1, 1)
    else:            rc = lib.mpc_beaver_matmul3(ctx, *[share3() for _ in range(6)], *s, f_public, 0)
    names = launches()
    opening = [n for n in names if "k_open_recode" in n]
    assert len(opening) <= 1
    return rc, names, int(opening[0].split("@")[1]) if opening else 0
'''


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    d = tmp_path_factory.mktemp("fake")
    return lambda body: fake_hip.run(d, CALLS + body)


def tiles(M, K, N, batch):
    """128 rows of one, 64 of two or 32 of four k blocks of the left operand, one k block by 128 columns of the right one."""
    up = lambda a, b: -(-a // b)
    kb = up(K, 16) + up(K, 16) % 2
    wide = kb if kb <= 2 else 4
    return batch * (up(M, 128 // wide) * up(kb, wide) + up(N, 128) * kb)


@pytest.mark.parametrize("parties", [2, 3])
def test_every_tile_of_a_small_call_has_a_workgroup(run, parties):
    """On a workspace of exactly the queried size; and the smallest workspace that a call accepts has no room for that."""
    shapes = [(1, 64, 10, 1), (1, 1, 2, 1), (13, 22, 8, 21), (2, 5, 58, 1), (11, 5, 297, 3), (2, 63, 455, 5), (3, 300, 130, 1)]
    r = run(f'''
for s in {shapes}:
    full, low = query({parties}, *s), 0
    high = full
    while high - low > 256:
        mid = (low + high) // 512 * 256
        rc, _, _ = product({parties}, mid, *s)
        assert rc in (0, -2), rc
        if rc == 0: high = mid
        else: low = mid
    result[str(s)] = product({parties}, full, *s), product({parties}, high, *s), full, high
''')
    less = 0
    for s in shapes:
        (rc, _, blocks), (rc_low, _, blocks_low), full, low = r[str(s)]
        assert rc == 0 and rc_low == 0
        assert blocks == tiles(*s), (s, blocks)
        assert blocks_low <= blocks and low <= full
        less += blocks_low < blocks
    assert less >= 4


def test_left_operand_with_a_public_right_one(run):
    """f public: the right planes are recoded in a launch of their own, and up to 2^20 words the left ones with them, behind
    the masking launch; a larger left operand opens in one launch ahead of it."""
    r = run('''
f = array(1 << 30)
for s in ((3, 6, 6, 1), (22, 52, 216, 55), (1024, 1024, 64, 1), (1024, 1025, 64, 1), (1467, 1038, 291, 1)):
    result[str(s)] = product(2, query(2, *s), *s, f_public=f)
    result[str(s) + " both"] = product(2, query(2, *s), *s)
''')
    for s in ((3, 6, 6, 1), (22, 52, 216, 55), (1024, 1024, 64, 1), (1024, 1025, 64, 1), (1467, 1038, 291, 1)):
        M, K, _, batch = s
        (rc, names, blocks), (rc_both, names_both, blocks_both) = r[str(s)], r[str(s) + " both"]
        assert rc == 0 and rc_both == 0
        assert (blocks > 0) == (M * K * batch > 1 << 20), (s, names)
        assert sum("k_sub_multi" in n for n in names) == (blocks == 0) and sum("k_recode" in n for n in names) == 1, names
        assert blocks_both > 0 and not any("k_sub_multi" in n or "k_recode" in n for n in names_both)


def test_input_gradient_with_a_secret_filter(run):
    """The filter is read in reverse tap order and recoded in a launch of its own: the same."""
    r = run('''
for B in (2, 65):
    g = (B, 16, 16, 32, 64, 3, 3, 1, 1)
    ws = lib.mpc_conv2d_grad_x_workspace_bytes(*g)
    assert lib.mpc_ctx_set_workspace(ctx, array(ws), ws) == 0
    rc = lib.mpc_conv2d_grad_x(ctx, *[share() for _ in range(6)], *g, None, 1, 1)
    result[B] = rc, launches()
''')
    for B in (2, 65):
        rc, names = r[str(B)]
        assert rc == 0
        assert any("k_open_recode" in n for n in names) == (B * 16 * 16 * 64 > 1 << 20), names


def test_im2col_of_few_channels(run):
    """Filter gradients of 3x3 filters: three units a thread from 8 channels on, with two to seven while the planes are small."""
    r = run('''
lib.mpc_conv2d_grad_w_workspace_bytes.restype = c_size_t; lib.mpc_conv2d_grad_w_workspace_bytes.argtypes = [c_int] * 9
lib.mpc_conv2d_grad_w.argtypes = [c_void_p] + [Share] * 6 + [c_int] * 9 + [c_void_p, c_int, c_int]
for B, HW, Cin in ((8, 32, 1), (32, 32, 2), (33, 32, 2), (32, 32, 3), (8, 112, 3), (8, 224, 7), (8, 224, 8), (1, 4, 200)):
    g = (B, HW, HW, Cin, 16, 3, 3, 1, 1)
    ws = lib.mpc_conv2d_grad_w_workspace_bytes(*g)
    assert lib.mpc_ctx_set_workspace(ctx, array(ws), ws) == 0
    rc = lib.mpc_conv2d_grad_w(ctx, *[share() for _ in range(6)], *g, None, 1, 1)
    names = launches()
    result["%d %d %d" % (B, HW, Cin)] = rc, sum("k_recode_im2col3_t" in n for n in names), sum("k_recode_im2col_t" in n for n in names)
''')
    three = {"8 32 1": 0, "32 32 2": 1, "33 32 2": 0, "32 32 3": 1, "8 112 3": 0, "8 224 7": 0, "8 224 8": 1, "1 4 200": 1}
    for k, (rc, with_three, with_one) in r.items():
        assert rc == 0 and (with_three, with_one) == (three[k], 1 - three[k]), (k, rc, with_three, with_one)


def test_every_tile_of_a_filter_gradients_right_operand_has_a_workgroup(run):
    """The output gradient alone opens in the launch: [B Ho Wo][Cout] words, a k block of 16 pixels a tile."""
    r = run('''
lib.mpc_conv2d_grad_w_workspace_bytes.restype = c_size_t; lib.mpc_conv2d_grad_w_workspace_bytes.argtypes = [c_int] * 9
lib.mpc_conv2d_grad_w.argtypes = [c_void_p] + [Share] * 6 + [c_int] * 9 + [c_void_p, c_int, c_int]
for HW, Cin in ((32, 1), (24, 2), (10, 1)):
    g = (1, HW, HW, Cin, 8, 3, 3, 1, 1)
    ws = lib.mpc_conv2d_grad_w_workspace_bytes(*g)
    assert lib.mpc_ctx_set_workspace(ctx, array(ws), ws) == 0
    assert lib.mpc_conv2d_grad_w(ctx, *[share() for _ in range(6)], *g, None, 1, 1) == 0
    result[HW] = [int(n.split("@")[1]) for n in launches() if "k_open_recode" in n]
''')
    for HW, blocks in r.items():
        kb = -(-int(HW) ** 2 // 16)
        assert blocks == [kb + kb % 2], (HW, blocks)


def test_operands_that_fill_few_of_their_tiles(run):
    """With more tiles than workgroups: long operands of few contiguous rows are opened by the separate kernels, others in one
    launch; three parties plain only after many rounds."""
    two = {(3, 9000, 4, 1): False, (3, 8000, 4, 1): False, (17, 3000, 8, 16): False, (3, 9000, 40, 1): True, (3, 4000, 4, 1): True,
           (3000, 2, 40, 16): True, (300, 3000, 300, 1): True}
    three = {(3, 40000, 4, 1): False, (3, 9000, 4, 1): True, (3000, 2, 40, 16): True, (3, 300, 4, 1): True}
    r = run(f'''
for s in {list(two)}: result["2 " + str(s)] = product(2, query(2, *s), *s)
for s in {list(three)}: result["3 " + str(s)] = product(3, query(3, *s), *s)
''')
    for n, cases in (("2 ", two), ("3 ", three)):
        for s, one in cases.items():
            rc, names, blocks = r[n + str(s)]
            assert rc == 0 and (blocks > 0) == one, (n, s, names)
