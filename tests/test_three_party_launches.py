"""Which GEMM launches a three-party product makes, on the CPU: the built library's host side on a stand-in for the HIP
runtime (fake_hip.cpp) that records the launched kernels.  Either one launch of the form with few tiles holds all parties,
or two launches hold two and one: whatever another thread sets mpc_set_gemm_small_tile to meanwhile, every call returns
MPC_OK and no other kernel is given three parties."""
import pytest

import fake_hip

PRODUCT = r'''
assert lib.mpc_ctx_set_exchange(ctx, 1) == 0
lib.mpc_matmul3_workspace_bytes.restype = c_size_t
lib.mpc_matmul3_workspace_bytes.argtypes = [c_int] * 4
lib.mpc_beaver_matmul3.argtypes = [c_void_p] + [Share3] * 6 + [c_int] * 4 + [c_void_p, c_int]

def product(M, K, N):
    """A call's arguments."""
    ws = lib.mpc_matmul3_workspace_bytes(M, K, N, 1)
    assert ws and lib.mpc_ctx_set_workspace(ctx, array(ws), ws) == 0
    return [Share3((c_void_p * 3)(*[array(8 * n) for _ in range(3)])) for n in (M * K, K * N, M * K, K * N, M * N, M * N)]

def call(shares, M, K, N):
    rc = lib.mpc_beaver_matmul3(ctx, *shares, M, K, N, 1, None, 0)
    return rc, [n for n in launches() if "gemm" in n]
'''


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    d = tmp_path_factory.mktemp("fake")
    return lambda body: fake_hip.run(d, PRODUCT + body)


def one_launch(names):
    return len(names) == 1 and "k_sliced_gemm" in names[0]


def test_few_tiles_take_one_launch_and_others_two(run):
    r = run('''
for shape in ((40, 1024, 33), (64, 64, 64), (2048, 256, 512)):
    result[str(shape)] = call(product(*shape), *shape)
lib.mpc_set_gemm_small_tile(0, 512)
result["off"] = call(product(40, 1024, 33), 40, 1024, 33)
''')
    assert all(rc == 0 for rc, _ in r.values()), r
    assert one_launch(r["(40, 1024, 33)"][1]) and one_launch(r["(64, 64, 64)"][1])
    for key in ("(2048, 256, 512)", "off"):
        assert sum("k_splitk" not in n for n in r[key][1]) == 2, r[key]


def test_outputs_over_addends(run):
    """Party 2 may store its output over c_0 or c_1 (parties 0 and 1 have read them by then): two launches.  Every party's
    output over its own c: a word is read by the thread that stores it, one launch."""
    r = run('''
shape = (40, 1024, 33)
for name, i, j, off in (("over c_0", 2, 0, 0), ("in c_1", 2, 1, 40), ("the end of c_0", 2, 0, 40 * 33 * 8 - 8), ("own c", 2, 2, 0), ("ahead of c_0", 2, 0, -40 * 33 * 8)):
    s = product(*shape)
    s[5].p[i] = s[4].p[j] + off
    result[name] = call(s, *shape)
''')
    assert all(rc == 0 for rc, _ in r.values()), r
    for name in ("over c_0", "in c_1", "the end of c_0"):
        assert len([n for n in r[name][1] if "k_splitk" not in n]) == 2, (name, r[name])
    assert one_launch(r["own c"][1]) and one_launch(r["ahead of c_0"][1])


def test_tuning_changed_by_another_thread_meanwhile(run):
    """40 x 1024 x 33 takes three slices and more on the larger tiles: the partial products of a third party have no room."""
    r = run('''
shares = product(40, 1024, 33)
kinds = {}
fake.fake_toggle_start(lib.mpc_set_gemm_small_tile, 0, 16, 512)
for _ in range(100000):
    rc, names = call(shares, 40, 1024, 33)
    key = "%d %s" % (rc, " ".join(names))
    kinds[key] = kinds.get(key, 0) + 1
fake.fake_toggle_stop()
result["kinds"] = kinds
''')
    for key, count in r["kinds"].items():
        rc, *names = key.split()
        names = [n for n in names if "k_splitk" not in n]
        assert rc == "0", f"{count} calls returned {rc} after {names}"
        assert one_launch(names) or len(names) == 2, f"{count} calls with three parties in {names}"
