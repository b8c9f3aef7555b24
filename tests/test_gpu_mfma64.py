"""The FP64 matrix-core kernel of N = 4 and 6 (variants "block" and "wave" of
the rotation route in FP64 and the compensated modes) against the oracle:
grids of a few cells, ragged tiles, media that begin and end inside a group of
sixteen cells, the boundary cell at a tile's edge, and rotation angles beyond
the short series.

err_E = max |E - E_oracle| / max |E_oracle|, err_pop = max |rho_aa - oracle|.
Tolerances: FP64 1e-10, single precision 1e-5 (the bars of the other kernels).
"""
import numpy as np
import pytest

from paper_1710_09799_amd import mln
from paper_1710_09799_amd import workloads as W

pytestmark = pytest.mark.gpu
TOL = {"fp64": 1e-10, "fp32c": 1e-5, "fp32cf": 1e-5}


def _errs(got, ref):
    e = np.concatenate([got["e_snap"].ravel(), got["probe"]])
    er = np.concatenate([ref["e_snap"].ravel(), ref["probe"]])
    err_p = np.max(np.abs(got["pop"] - ref["pop"])) if ref["pop"].size else 0.0
    return np.max(np.abs(e - er)) / np.max(np.abs(er)), err_p


@pytest.fixture(scope="module")
def refs(orc):
    cache = {}

    def get(key, problem, snap):
        if key not in cache:
            cache[key] = orc.run(problem, snap_every=snap)
        return cache[key]
    return get


@pytest.mark.parametrize("n", [4, 6])
@pytest.mark.parametrize("precision", ["fp64", "fp32c", "fp32cf"])
@pytest.mark.parametrize("tile,k", [(64, 7), (128, 24), (192, 5), (256, 60)])
@pytest.mark.parametrize("nx,med", [(3, (1, 2)), (101, None), (417, (63, 303)), (209, (5, 5))])
def test_mfma64_tiles(refs, n, precision, tile, k, nx, med):
    p = W.random_problem(n, 40 + n, nx=nx, nt=150, med=med)
    print(f"[case] mfma64 n={n} {precision} tile={tile} k={k} nx={nx} med={med}", flush=True)
    got = mln.run(p, precision=precision, snap_every=33, variant="block", tile=tile, steps_per_launch=k)
    ee, ep = _errs(got, refs((n, nx, med), p, 33))
    assert ee < TOL[precision] and ep < TOL[precision], (ee, ep)


@pytest.mark.parametrize("n", [4, 6])
@pytest.mark.parametrize("scale", [30.0, 1000.0, 30000.0])
def test_mfma64_wide_angles(refs, n, scale):
    p = W.random_problem(n, 60 + n, nx=150, nt=120)
    p.source.amplitude *= scale
    got = mln.run(p, precision="fp64", snap_every=30, variant="block", tile=64, steps_per_launch=16)
    ee, ep = _errs(got, refs((n, scale), p, 30))
    print(f"[case] mfma64 angles n={n} scale={scale} err_E={ee:.1e} err_pop={ep:.1e}", flush=True)
    assert ee < 1e-10 and ep < 1e-10, (ee, ep)


@pytest.mark.parametrize("n", [4, 6])
@pytest.mark.parametrize("precision", ["fp64", "fp32c", "fp32cf"])
def test_mfma64_any_boundary_cell_and_chunks(refs, n, precision):
    """The boundary cell at different places of a tile and of a group; a run
    in uneven chunks gives the bits of the whole run."""
    for nx in range(224, 224 + 34, 3):
        p = W.random_problem(n, nx, nx=nx, nt=100)
        s = mln.Solver(p, precision=precision, snap_every=50, variant="block", tile=64, steps_per_launch=8)
        a = {k: v.cpu().numpy().copy() for k, v in s.run().items()}
        s.reset()
        for k in (1, 37, 9):
            s.step(k)
        b = {k: v.cpu().numpy() for k, v in s.run().items()}
        s.close()
        for k in a:
            assert np.array_equal(a[k], b[k]), (nx, k)
        ee, ep = _errs(a, refs((n, "edge", nx), p, 50))
        assert ee < TOL[precision] and ep < TOL[precision], (nx, ee, ep)


@pytest.mark.parametrize("n", [4, 6])
def test_mfma64_automatic_shape(refs, n):
    """The automatic shape, also where a compute unit takes several tiles."""
    for nx in (700, 60000):
        p = W.random_problem(n, 9, nx=nx, nt=64, med=(50, nx - 20))
        s = mln.Solver(p, snap_every=32)
        assert s.config()["variant"] == "block"
        ee, ep = _errs({k: v.cpu().numpy() for k, v in s.run().items()}, refs((n, "auto", nx), p, 32))
        s.close()
        assert ee < 1e-10 and ep < 1e-10, (nx, ee, ep)
