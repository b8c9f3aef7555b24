"""The compensated FP32 state of the kernels that step it in FP64 and round it to
a pair of floats in every step (csrc/float_pair.hpp)."""
import numpy as np
import pytest

from paper_1710_09799_amd import mln
from paper_1710_09799_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["lane2", "lane3", "mfma4", "mfma6", "tmz2", "tmz3"])
def test_compensated_state_does_not_drift(kind):
    """A medium without a field, 20000 steps, against FP64.  To the nearest of 49
    bits the roundings, at most 2^-50 of values up to 1, make a random walk, the
    same in every cell: 8 sqrt(nt) 2^-50 = 1e-12.  Rounding towards zero to 48
    bits adds up to nt 2^-49 = 4e-11; plain FP32 walks in steps of 2^-25."""
    n, nt = int(kind[-1]), 20000
    tmz = kind[:3] == "tmz"
    p = W.random_problem_2d(n, 3, nx=40, ny=6, nt=nt) if tmz else W.random_problem(n, 3, nx=90, nt=nt)
    p.source.amplitude = 0.0
    p.medium.density = 1e-12  # no field of its own either
    run = mln.tmz_run if tmz else mln.run
    kw = {} if tmz else dict(variant="block", tile=64, steps_per_launch=16)
    pop = {q: run(p, precision=q, snap_every=nt // 10, **kw)["pop"] for q in ("fp64", "fp32c", "fp32")}
    err = {q: np.max(np.abs(pop[q] - pop["fp64"])) for q in ("fp32c", "fp32")}
    print(f"[case] drift {kind} fp32c {err['fp32c']:.1e} fp32 {err['fp32']:.1e}", flush=True)
    tol = 8 * np.sqrt(nt) * 2.0**-50
    assert err["fp32c"] < tol < err["fp32"], (err, tol)
