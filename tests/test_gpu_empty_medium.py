"""A medium of no cells (med_begin == med_end, or an empty rectangle) in every
solver of the Yee grid: the fields of the oracle, and nothing recorded."""
import numpy as np
import pytest

from paper_1710_09799_amd import mln
from paper_1710_09799_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,variant,precision", [(2, "quad", "fp64"), (3, "quad_mfma", "fp32c"), (3, "block", "fp64"),
                                                 (2, "block", "fp32cf"), (3, "wave", "fp64"), (4, "block", "fp64"),
                                                 (6, "block", "fp32c"), (4, "quad", "bf16x6"), (6, "block", "bf16x6"),
                                                 (2, "stream", "fp64")])
@pytest.mark.parametrize("at", [1, 64, 129])
def test_line(orc, n, variant, precision, at):
    p = W.random_problem(n, 8, nx=130, nt=250, med=(at, at))
    print(f"[case] empty medium n={n} {variant} {precision} at {at}", flush=True)
    got, ref = mln.run(p, precision=precision, snap_every=50, variant=variant), orc.run(p, snap_every=50)
    assert got["pop"].shape == (5, n, 0)
    for k in ("probe", "e_snap"):
        assert np.max(np.abs(got[k] - ref[k])) < (1e-12 if precision == "fp64" else 1e-5) * np.max(np.abs(ref["e_snap"]))


@pytest.mark.parametrize("n", [2, 3, 4])
@pytest.mark.parametrize("rect", [(1, 1, 0, 20), (64, 64, 3, 9), (10, 70, 5, 5)])
def test_tmz(orc, n, rect):
    p = W.random_problem_2d(n, 8, nx=90, ny=20, nt=150, rect=rect)
    print(f"[case] empty medium tmz n={n} {rect}", flush=True)
    got, ref = mln.tmz_run(p, snap_every=50), orc.run2d(p, snap_every=50)
    for k in ("probe", "e_snap"):
        assert np.max(np.abs(got[k] - ref[k])) < 1e-12 * np.max(np.abs(ref["e_snap"]))


def test_batch(orc):
    probs = [W.random_problem(2 + i % 2, 20 + i, nx=70 + 40 * i, nt=200, med=(5, 5) if i % 3 else None) for i in range(5)]
    b = mln.Batch(probs, precision="fp64", snap_every=100)
    for p, o in zip(probs, b.run()):
        ref = orc.run(p, snap_every=100)
        assert np.max(np.abs(o["e_snap"].cpu().numpy() - ref["e_snap"])) < 1e-12 * np.max(np.abs(ref["e_snap"]))
    b.close()
