"""pair_exact (csrc/float_pair.hpp), compiled for the host: the nearest value of
49 bits, which a pair of floats holds, without a drift."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1710_09799_amd", "csrc")
SHIM = """
#include "float_pair.hpp"
extern "C" void pairs(long n, const double *x, double *r) {
  for (long i = 0; i < n; ++i) r[i] = mln::pair_exact(x[i]);
}
"""


@pytest.fixture(scope="module")
def pair_exact(tmp_path_factory):
    d = tmp_path_factory.mktemp("float_pair")
    src, so = d / "shim.cpp", d / "shim.so"
    src.write_text(SHIM)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I" + CSRC, str(src), "-o", str(so)])
    L = ctypes.CDLL(str(so))

    def call(x):
        x = np.ascontiguousarray(x, dtype=np.float64)
        r = np.empty_like(x)
        L.pairs(ctypes.c_long(x.size), ctypes.c_void_p(x.ctypes.data), ctypes.c_void_p(r.ctypes.data))
        return x, r
    return call


def _values(lo, hi):
    rng = np.random.default_rng(17)
    x = np.exp2(rng.uniform(lo, hi, 100000)) * rng.choice([-1.0, 1.0], 100000)
    k = np.arange(1, 4000, dtype=np.float64)
    e = np.exp2(float(int((lo + hi) / 2)))
    return np.concatenate([x, e * (1 + k * 2.0**-52), e * (2 - k * 2.0**-52), -e * (1 + k * 2.0**-52)])


def _unit(x):
    """The last place of 49 bits."""
    return np.ldexp(1.0, np.frexp(x)[1] - 49)


@pytest.mark.parametrize("lo,hi", [(-3, 1), (-60, -20), (-100, -90), (-140, -100), (20, 100)])
def test_nearest_and_held_by_a_pair(pair_exact, lo, hi):
    x, r = pair_exact(_values(lo, hi))
    unit = np.maximum(_unit(x), 2.0**-149)
    assert np.array_equal(r, np.rint(x / unit) * unit)  # exact: powers of two, ties to even
    h = r.astype(np.float32)
    low = (r - h.astype(np.float64)).astype(np.float32)
    assert np.array_equal(h.astype(np.float64) + low.astype(np.float64), r)


def test_no_drift(pair_exact):
    """The mean of the rounding towards larger magnitudes, in units of the last
    place: 1e5 roundings of at most half a unit, 5 standard deviations."""
    x, r = pair_exact(_values(-3, 1)[:100000])
    unit = _unit(x)
    assert abs(np.mean((np.abs(r) - np.abs(x)) / unit)) < 5 * 0.29 / np.sqrt(1e5)


def test_special_values(pair_exact):
    _, r = pair_exact([0.0, -0.0, np.inf, -np.inf, np.nan, 1e-300, 5e-324])
    assert r[0] == 0 and r[1] == 0 and r[2] == np.inf and r[3] == -np.inf and np.isnan(r[4]) and r[5] == 0 and r[6] == 0
