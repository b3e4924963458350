"""The rule that keeps a call from running as one launch when an output shares memory with an input (csrc/overlap.h),
compiled on the host and compared with the byte sets themselves over all small placements."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2209_13643_amd", "csrc")
SOURCE = r'''
#include "overlap.h"
extern "C" int apart(size_t o, size_t on, int ob, size_t i, size_t in_, int ib, int same)
{
    Spans<1> out, in;
    if (ob) out.bytes((const void*)o, on); else out.words((const void*)o, on);
    if (ib) in.bytes((const void*)i, in_); else in.words((const void*)i, in_);
    return outputs_apart(out, in, same != 0);
}
'''


@pytest.fixture(scope="module")
def apart(tmp_path_factory):
    d = tmp_path_factory.mktemp("overlap")
    (d / "o.cpp").write_text(SOURCE)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(d / "o.cpp"), "-o", str(d / "o.so")])
    f = ctypes.CDLL(str(d / "o.so")).apart
    f.argtypes = [ctypes.c_size_t, ctypes.c_size_t, ctypes.c_int, ctypes.c_size_t, ctypes.c_size_t, ctypes.c_int, ctypes.c_int]
    return f


@pytest.mark.parametrize("same", [0, 1])
def test_against_the_byte_sets(apart, same):
    for ob in (0, 1):
        for ib in (0, 1):
            for on in (1, 3):
                for n in (1, 2, 5):
                    for o in list(range(64, 72)) + [80, 104]:
                        for i in list(range(40, 100, 4)) + [65, 67]:
                            a = set(range(o, o + on * (1 if ob else 8)))
                            b = set(range(i, i + n * (1 if ib else 8)))
                            want = not (a & b) or (same and o == i and ob == ib)
                            assert bool(apart(o, on, ob, i, n, ib, same)) == bool(want), (o, on, ob, i, n, ib, same)


def test_absent_arrays_do_not_count(apart):
    assert apart(0, 5, 0, 64, 5, 0, 0) and apart(64, 5, 1, 0, 100, 0, 1)
