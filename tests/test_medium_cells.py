"""Where a run of cells meets the medium (csrc/medium_cells.hpp), compiled for
the host: kernels whose loads no lane skips read the state at
nearest_medium(), which has to stay inside a row of the state arrays, also
for an empty medium (med_begin == med_end), where rows hold one element."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1710_09799_amd", "csrc")
SHIM = """
#include "medium_cells.hpp"
extern "C" int meets(long i0, long n, long mb, long me) { return mln::meets_medium(i0, n, mb, me); }
extern "C" long nearest(long i, long mb, long me) { return mln::nearest_medium(i, mb, me); }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("medium_cells")
    src, so = d / "shim.cpp", d / "shim.so"
    src.write_text(SHIM)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I" + CSRC, str(src), "-o", str(so)])
    L = ctypes.CDLL(str(so))
    L.nearest.restype = ctypes.c_long
    for f in (L.meets, L.nearest):
        f.argtypes = [ctypes.c_long] * (4 if f is L.meets else 3)
    return L


# empty, one cell, a few, in the middle and at both ends of a 40-cell grid
@pytest.mark.parametrize("mb,me", [(1, 1), (5, 5), (39, 39), (1, 2), (38, 39), (16, 17), (1, 39), (15, 33)])
def test_against_the_cells(lib, mb, me):
    cells = range(mb, me)
    for i in range(-70, 110):
        col = lib.nearest(i, mb, me)
        assert 0 <= col < max(1, me - mb), (i, col)
        if cells:
            assert abs(i - (mb + col)) == min(abs(i - c) for c in cells), (i, col)
        for n in (1, 16, 32, 64):
            assert bool(lib.meets(i, n, mb, me)) == any(i <= c < i + n for c in cells), (i, n)
