"""Several steps per launch on the 2-D TMz grid (N = 2, 3) against the oracle:
grids narrower and lower than a tile (rows wrap more than once), ragged tiles
in both directions, media that begin and end inside tiles, recordings in the
middle of a launch, launches cut by uneven stepping, and the Mur column in any
place of a tile.  Bars as in test_gpu_tmz.py: FP64 1e-10, single precision 1e-5.
"""
import numpy as np
import pytest

from paper_1710_09799_amd import mln
from paper_1710_09799_amd import workloads as W

pytestmark = pytest.mark.gpu
TOL = {"fp64": 1e-10, "fp32c": 1e-5, "fp32": 1e-5}


def _errs(got, ref):
    e = np.concatenate([got["e_snap"].ravel(), got["probe"].ravel()])
    er = np.concatenate([ref["e_snap"].ravel(), ref["probe"].ravel()])
    err_p = np.max(np.abs(got["pop"] - ref["pop"])) if ref["pop"].size else 0.0
    scale = np.max(np.abs(er)) * np.sqrt(W.EPS0 / W.MU0)
    err_h = max(np.max(np.abs(got["hx"] - ref["hx"])), np.max(np.abs(got["hy"][:, :-1] - ref["hy"][:, :-1])))
    return np.max(np.abs(e - er)) / np.max(np.abs(er)), err_p, err_h / scale


@pytest.mark.parametrize("n", [2, 3])
@pytest.mark.parametrize("precision", ["fp64", "fp32c", "fp32"])
@pytest.mark.parametrize("nx,ny,rect", [(3, 1, (1, 2, 0, 1)), (20, 3, (4, 19, 1, 2)), (64, 5, None),
                                        (119, 40, (30, 90, 0, 40)), (200, 67, (1, 199, 11, 50)),
                                        (131, 97, (60, 61, 5, 90))])
def test_tmz_tiles(orc, n, precision, nx, ny, rect):
    p = W.random_problem_2d(n, 70 + n, nx=nx, ny=ny, nt=150, rect=rect)
    print(f"[case] tmz tiles n={n} {precision} {nx}x{ny} {rect}", flush=True)
    ref = orc.run2d(p, snap_every=37)
    got = mln.tmz_run(p, precision=precision, snap_every=37)
    errs = _errs(got, ref)
    assert max(errs) < TOL[precision], errs


def test_tmz_uneven_steps_and_any_mur_column(orc):
    """Chunks of a run equal the whole run bit for bit, on widths that put
    the Mur column at different places of the last tile."""
    for nx in range(100, 112):
        p = W.random_problem_2d(3, nx, nx=nx, ny=20, nt=90, rect=(2, nx - 1, 0, 20))
        ref = orc.run2d(p, snap_every=30)
        s = mln.Tmz(p, snap_every=30)
        a = {k: v.cpu().numpy().copy() for k, v in s.run().items()}
        a["ez"], a["hx"], a["hy"] = s.fields()
        s.reset()
        for k in (1, 2, 13, 50):
            s.step(k)
        b = {k: v.cpu().numpy().copy() for k, v in s.run().items()}
        s.reset()
        for _ in range(90):
            s.step(1)
        c = {k: v.cpu().numpy() for k, v in s.run().items()}
        s.close()
        for k in b:
            assert np.array_equal(a[k], b[k]) and np.array_equal(a[k], c[k]), (nx, k)
        errs = _errs(a, ref)
        assert max(errs) < 1e-10, (nx, errs)


def test_tmz_large_tiles_agree_with_oracle(orc):
    """A grid whose shape takes the tallest tiles."""
    p = W.random_problem_2d(3, 90, nx=1500, ny=401, nt=40, rect=(5, 1400, 20, 390))
    print("[case] tmz large tiles", flush=True)
    ref = orc.run2d(p, snap_every=20)
    for precision in ("fp64", "fp32c", "fp32"):
        errs = _errs(mln.tmz_run(p, precision=precision, snap_every=20), ref)
        assert max(errs) < TOL[precision], (precision, errs)
