"""The k blocks that workgroups of the tile recoder take (csrc/recode_tiles.h, compiled on the host): every block of a
plane once, none past its end, also for the grid indices a set gets from a larger set of the same launch."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2209_13643_amd", "csrc")
SOURCE = r'''
#include "recode_tiles.h"
extern "C" unsigned count(int ntaps, int kb_tap, int kb_total) { return recode_tile_count(ntaps, kb_tap, kb_total); }
extern "C" void tile(int ntaps, int kb_tap, int kb_total, unsigned by, int* out)
{
    const RecodeTile t = recode_tile(ntaps, kb_tap, kb_total, by);
    out[0] = t.tap; out[1] = t.kb0; out[2] = t.kb_lim; out[3] = t.zero;
}
'''


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("tiles")
    (d / "t.cpp").write_text(SOURCE)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(d / "t.cpp"), "-o", str(d / "t.so")])
    L = ctypes.CDLL(str(d / "t.so"))
    L.count.restype = ctypes.c_uint
    return L


@pytest.mark.parametrize("ntaps", [1, 2, 3, 4, 9, 25])
def test_every_block_once_and_none_past_the_plane(lib, ntaps):
    out = (ctypes.c_int * 4)()
    for kb_tap in (1, 2, 3, 4, 5, 7, 8, 9, 16, 33):
        if ntaps > 1 and kb_tap < 2:
            continue                                     # such filters take the other recoder
        kb_total = (ntaps * kb_tap + 1) // 2 * 2         # whole pairs of blocks
        taken = {}
        for by in range(lib.count(ntaps, kb_tap, kb_total) + 3 * kb_total + 40):
            lib.tile(ntaps, kb_tap, kb_total, by, out)
            tap, kb0, lim, zero = out[:]
            for kb in range(kb0, min(kb0 + 4, lim)):
                block = tap * kb_tap + kb
                assert block < kb_total, (kb_tap, by, block, kb_total)
                assert block not in taken, (kb_tap, by, block)
                assert zero == (block >= ntaps * kb_tap and ntaps > 1)
                taken[block] = by
        assert sorted(taken) == list(range(kb_total))
        assert all(by < lib.count(ntaps, kb_tap, kb_total) for by in taken.values())
