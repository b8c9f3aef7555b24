"""Rotation angles far beyond the short series, in the kernels that evaluate
them with wide_angle.hpp.

FP32 against the oracle: the product theta E and E itself carry a few units of
2^-24 relative, so an angle of a rad is off by about 4 a 2^-24 in a step and the
populations by that per step: bar nt 4 (1 + a) 2^-24.  Angles of 1e8 rad (FP32)
and 1e17 rad (FP64) say nothing about the state (from three levels on not even
that it is positive: the angles' roundings are whole turns), but a rotation
keeps the Bloch vector's length, so the populations stay within 1/N +- (1 - 1/N)
to rounding, a few 2^-24 (2^-53) per step."""
import numpy as np
import pytest

from paper_1710_09799_amd import mln
from paper_1710_09799_amd import workloads as W

pytestmark = pytest.mark.gpu
NT = 120


def _step_angle(p, e):
    """The largest rotation angle of a step at the field e."""
    ev = np.linalg.eigvalsh(p.medium.dipole)
    return (ev[-1] - ev[0]) * e * p.grid.dt / W.HBAR


@pytest.mark.parametrize("n", [2, 3])
@pytest.mark.parametrize("scale", [30.0, 1000.0, 30000.0])
def test_fp32_wide_angles(orc, n, scale):
    p = W.random_problem(n, 60 + n, nx=150, nt=NT)
    p.source.amplitude *= scale
    ref = orc.run(p, snap_every=30)
    a = _step_angle(p, np.max(np.abs(ref["e_snap"])))
    got = mln.run(p, precision="fp32", snap_every=30, variant="block", tile=64, steps_per_launch=16)
    err = np.max(np.abs(got["pop"] - ref["pop"]))
    print(f"[case] fp32 angles n={n} scale={scale} a={a:.1f} err_pop={err:.1e}", flush=True)
    assert err < NT * 4 * (1 + a) * 2.0**-24, err


@pytest.mark.parametrize("precision,scale", [("fp32", 1e10), ("fp64", 1e19), ("fp32c", 1e10)])
@pytest.mark.parametrize("kind", ["lane2", "lane3", "mfma4", "mfma6", "tmz2", "tmz3"])
def test_huge_angles_keep_the_length(kind, precision, scale):
    n = int(kind[-1])
    if kind[:3] == "tmz":
        p = W.random_problem_2d(n, 70 + n, nx=80, ny=20, nt=NT)
    else:
        p = W.random_problem(n, 60 + n, nx=150, nt=NT)
    p.source.amplitude *= scale
    if kind[:3] == "tmz":
        pop = mln.tmz_run(p, precision=precision, snap_every=30)["pop"]
    else:
        pop = mln.run(p, precision=precision, snap_every=30, variant="block", tile=64, steps_per_launch=16)["pop"]
    tol = NT * 40 * (2.0**-53 if precision == "fp64" else 2.0**-24)
    print(f"[case] huge angles {kind} {precision} {pop.min():.3e} {pop.max():.6f}", flush=True)
    assert np.isfinite(pop).all() and pop.min() > 2 / n - 1 - tol and pop.max() < 1 + tol, (pop.min(), pop.max())
    assert np.max(np.abs(pop.sum(axis=1) - 1)) < tol
