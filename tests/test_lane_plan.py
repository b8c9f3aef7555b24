"""The automatic choice between four lanes per cell and one wavefront per tile
(csrc/lane_plan.hpp), compiled for the host: the kernel that measured faster, at
sizes where the two differ by more than a few percent."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1710_09799_amd", "csrc")
SHIM = """
#include "lane_plan.hpp"
extern "C" long min_cells(int n, int fp32, int comp) { return mln::lane_min_cells(n, fp32, comp); }
extern "C" int fits(unsigned long bytes, unsigned long free_bytes) { return mln::second_buffer_fits(bytes, free_bytes); }
extern "C" void plan(int n, int fp32, int bytes, long nx, int cus, int *w, int *k) {
  const mln::LanePlan p = mln::lane_plan(n, fp32, bytes, nx, cus);
  *w = p.W; *k = p.K;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("lane_plan")
    src, so = d / "shim.cpp", d / "shim.so"
    src.write_text(SHIM)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I" + CSRC, str(src), "-o", str(so)])
    L = ctypes.CDLL(str(so))
    L.min_cells.restype = ctypes.c_long
    return L


# us per step, one wavefront per tile / four lanes per cell
MEASURED = {
    (2, "fp64"): {3000: (0.55, 0.49), 8000: (0.57, 0.51), 14000: (0.65, 0.54), 20000: (0.65, 0.59), 26000: (0.65, 0.77)},
    (2, "fp32"): {12000: (0.54, 0.43), 20000: (0.59, 0.48), 25000: (0.56, 0.69), 36000: (0.56, 0.60)},
    (2, "fp32c"): {3000: (0.58, 0.52), 8000: (0.59, 0.53), 14000: (0.69, 0.56), 20000: (0.70, 0.62), 25000: (0.71, 0.85),
                   36000: (0.74, 0.88)},
    (3, "fp64"): {20000: (0.92, 0.73), 22500: (0.92, 0.81), 24000: (0.90, 0.93), 36000: (0.99, 1.06)},
    (3, "fp32"): {33000: (0.88, 0.77), 36000: (0.88, 0.79), 40000: (0.90, 0.94), 50000: (0.95, 1.05)},
    (3, "fp32c"): {40000: (1.19, 1.12), 75000: (1.49, 1.72), 90000: (1.51, 1.84)},
}


@pytest.mark.parametrize("n,precision", sorted(MEASURED))
def test_faster_kernel_is_chosen(lib, n, precision):
    least = lib.min_cells(n, precision == "fp32", precision == "fp32c")
    for nx, (wave, quad) in MEASURED[(n, precision)].items():
        assert (nx >= least) == (wave < quad), (nx, least)


@pytest.mark.parametrize("state", [10**6, 5 * 10**7, 10**9, 3 * 10**10, 10**11, 2 * 10**11])
def test_second_buffer_leaves_room(lib, state):
    """Handles of one state each on a card of 288 GB: the second buffers never
    take more than an eighth of what is free, and handles whose states would
    have filled the card still find seven eighths of it."""
    lib.fits.argtypes = [ctypes.c_ulong] * 2
    free, handles = 288 * 10**9, 0
    while free >= state and handles < 10000:
        free -= state
        handles += 1
        if lib.fits(state, free):
            assert 8 * state <= free
            free -= state
    assert free < state or handles == 10000
    alone = min(10000, 288 * 10**9 // state)
    if 9 * state > 288 * 10**9:  # a state beyond an eighth of the rest: as many as without the rule
        assert handles == alone
