"""A two-party ReLU on a workspace of exactly the queried size, default exchange, on the CPU: the launches its calls make on a
stand-in for the HIP runtime.  Up to 2^18 elements the queried size holds the buffers of the one launch that does all; the
size that the launch sequence alone needs is accepted as well."""
import pytest

import fake_hip

RELU = r'''
class Material(ctypes.Structure):
    _fields_ = [("p", c_void_p * 18)]
two = c_void_p * 2
for q in ("mpc_relu_workspace_bytes", "mpc_relu_msb_workspace_bytes", "mpc_relu_packed_words"):
    getattr(lib, q).restype = c_size_t; getattr(lib, q).argtypes = [c_size_t]
for f in ("mpc_relu", "mpc_relu_msb"):
    getattr(lib, f).argtypes = [c_void_p, Share, ctypes.POINTER(Material), Share, c_size_t, c_int, c_void_p, c_void_p]
SIZES = list(range(1, 301)) + [511, 512, 513, 4097, 65535, 65536, 65537, 65536 + 129, 131072, 131073, 200001, 262143, 262144, 262145]

def relu(n, packed, ws):
    assert lib.mpc_ctx_set_workspace(ctx, array(ws), ws) == 0
    mat = Material((c_void_p * 18)(*[array(8 * 16 * n) for _ in range(18)]))
    share = lambda: Share(two(array(8 * n), array(8 * n)))
    rc = (lib.mpc_relu_msb if packed else lib.mpc_relu)(ctx, share(), mat, share(), n, 0, None, None)
    return rc, launches()

def query(n, packed):
    return (lib.mpc_relu_msb_workspace_bytes if packed else lib.mpc_relu_workspace_bytes)(n)
'''


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    d = tmp_path_factory.mktemp("fake")
    return lambda body: fake_hip.run(d, RELU + body)


@pytest.mark.parametrize("packed", [0, 1])
def test_the_queried_workspace_holds_the_one_launch(run, packed):
    r = run(f'''
for n in SIZES:
    result[n] = relu(n, {packed}, query(n, {packed}))
''')
    for n, (rc, names) in r.items():
        assert rc == 0, (n, rc)
        if int(n) <= 1 << 18:
            assert len(names) == 1 and "k_relu_fused" in names[0], (n, names)
        else:
            assert len(names) > 10 and not any("k_relu_fused" in k for k in names), (n, names)


def sequence_bytes(n):
    """What the launch sequence keeps of a whole-word call's n elements: four rows sent and received, G and P, three rows of bytes."""
    up = lambda b: (b + 255) // 256 * 256
    return 2 * (2 * up(32 * n) + 2 * up(n) + 2 * up(8 * n) + up(n))


def test_the_earlier_workspace_is_enough(run):
    """The larger of the launch sequence's arrays and the buffers of the remote-store launch (two per workgroup of 64 elements,
    four rows of 64 words): such a call runs launch by launch where the copies' buffers do not fit."""
    sizes = (1, 20, 32, 33, 64, 65, 70, 88, 89, 129, 136, 137)
    r = run(f'''
for n, ws in {[(n, max(sequence_bytes(n), (n + 63) // 64 * 2 * 4 * 64 * 8)) for n in sizes]}:
    result[n] = relu(n, 0, ws), relu(n, 0, ws - 256)[0], ws
''')
    for n, ((rc, names), less, ws) in r.items():
        fits = ws >= (int(n) + 63) // 64 * 4 * 4 * 64 * 8
        assert rc == 0 and less == -2, (n, rc, less)
        assert (len(names) == 1) == fits, (n, names)
