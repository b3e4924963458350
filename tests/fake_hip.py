"""Runs calls of the built library's host side on a stand-in for the HIP runtime (fake_hip.cpp), in a process of its own:
nothing is executed, and the launched kernels' names and grids come back.  Used by tests that ask which launches a call makes."""
import json
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))

# The library is used through ctypes alone: a process that has loaded the real runtime's users first would not do.
CLIENT = r'''
import ctypes, json, sys
from ctypes import c_int, c_size_t, c_void_p
fake = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[2])

class Share(ctypes.Structure):
    _fields_ = [("p", c_void_p * 2)]

class Share3(ctypes.Structure):
    _fields_ = [("p", c_void_p * 3)]

lib.mpc_ctx_set_workspace.argtypes = [c_void_p, c_void_p, c_size_t]
lib.mpc_ctx_set_exchange.argtypes = [c_void_p, c_int]
fake.fake_launches.restype = c_size_t
text = ctypes.create_string_buffer(1 << 16)

def launches():
    """Kernels launched since the last call of this, each as name@workgroups."""
    fake.fake_launches(text, len(text))
    return text.value.decode().split()

ctx = c_void_p()
assert lib.mpc_ctx_create_single_queue(ctypes.byref(ctx), 0, 16) == 0
at = 1 << 40
def array(nbytes):
    """The address of an array at a place of its own; nothing reads it."""
    global at
    a, at = at, at + (nbytes + 4095) // 4096 * 4096
    return a

result = {}
'''


def run(tmp, body):
    """The value of `result` after `body` has run behind CLIENT."""
    from paper_2209_13643_amd import mpc
    if not os.path.exists(mpc.LIB_PATH):
        import __graft_entry__
        __graft_entry__.build()
    so = str(tmp / "fake_hip.so")
    if not os.path.exists(so):
        subprocess.check_call(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-pthread", os.path.join(HERE, "fake_hip.cpp"), "-o", so])
    out = subprocess.run([sys.executable, "-c", CLIENT + body + "\nprint(json.dumps(result))", so, mpc.LIB_PATH],
                         capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stderr[-2000:]
    return json.loads(out.stdout.splitlines()[-1])
