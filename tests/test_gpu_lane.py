"""The one-wavefront tile kernel (variant "block" with plain fields: tiles of
64 and 128 cells always, of 192 and 256 cells from three per compute unit on)
against the oracle: tiles with ragged ends, media that begin and end inside a
tile, halos that are no multiple of the cells per lane, and rotation angles
beyond the short series.

err_E = max |E - E_oracle| / max |E_oracle|, err_pop = max |rho_aa - oracle|.
Tolerances: FP64 1e-10, single precision 1e-5 (the bars of the other kernels).
"""
import numpy as np
import pytest

from paper_1710_09799_amd import mln
from paper_1710_09799_amd import workloads as W

pytestmark = pytest.mark.gpu
TOL = {"fp64": 1e-10, "fp32c": 1e-5, "fp32": 1e-5}


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


@pytest.mark.parametrize("n", [2, 3])
@pytest.mark.parametrize("precision", ["fp64", "fp32c", "fp32"])
@pytest.mark.parametrize("tile,k", [(64, 7), (64, 28), (128, 15), (128, 24)])
@pytest.mark.parametrize("nx,med", [(3, (1, 2)), (65, None), (208, (63, 130)), (417, (5, 5))])
def test_lane_tiles(refs, n, precision, tile, k, nx, med):
    p = W.random_problem(n, 40 + n, nx=nx, nt=200, med=med)
    print(f"[case] lane n={n} {precision} tile={tile} k={k} nx={nx} med={med}", flush=True)
    got = mln.run(p, precision=precision, snap_every=33, variant="block", tile=tile, steps_per_launch=k)
    ee, ep = _errs(got, refs((n, nx, med), p, 33))
    assert ee < TOL[precision] and ep < TOL[precision], (ee, ep)


@pytest.mark.parametrize("n", [2, 3])
@pytest.mark.parametrize("precision", ["fp64", "fp32c", "fp32"])
@pytest.mark.parametrize("tile,k", [(192, 90), (256, 121)])
def test_lane_wide_tiles(refs, n, precision, tile, k):
    """Three and four cells per lane: enough tiles by narrow owned parts."""
    nx = 11003
    p = W.random_problem(n, 50 + n, nx=nx, nt=130, med=(70, nx - 131))
    print(f"[case] lane n={n} {precision} tile={tile} k={k}", flush=True)
    got = mln.run(p, precision=precision, snap_every=65, variant="block", tile=tile, steps_per_launch=k)
    ee, ep = _errs(got, refs((n, "wide"), p, 65))
    assert ee < TOL[precision] and ep < TOL[precision], (ee, ep)


@pytest.mark.parametrize("n", [2, 3])
@pytest.mark.parametrize("scale", [30.0, 1000.0, 30000.0])
def test_lane_wide_angles(refs, n, scale):
    """Fields that turn a cell by up to about 1/4, 10 and 300 rad per step."""
    p = W.random_problem(n, 60 + n, nx=150, nt=120)
    p.source.amplitude *= scale
    got = mln.run(p, precision="fp64", snap_every=30, variant="block", tile=64, steps_per_launch=16)
    ee, ep = _errs(got, refs((n, scale), p, 30))
    print(f"[case] lane angles n={n} scale={scale} err_E={ee:.1e} err_pop={ep:.1e}", flush=True)
    assert ee < 1e-10 and ep < 1e-10, (ee, ep)


@pytest.mark.parametrize("precision", ["fp64", "fp32c"])
def test_lane_automatic_choice_and_chunks(precision):
    """A grid beyond the crossover takes the kernel by itself and agrees with
    the four-lane kernel; stepping in uneven chunks changes nothing."""
    p = W.three_level(nx=45000, nt=300)
    s = mln.Solver(p, precision=precision, snap_every=100)
    assert s.config()["variant"] == "block"
    a = {k: v.cpu().numpy().copy() for k, v in s.run().items()}
    s.reset()
    for k in (1, 37, 100, 162):
        s.step(k)
    b = {k: v.cpu().numpy() for k, v in s.run().items()}
    for k in a:
        assert np.array_equal(a[k], b[k]), k
    s.close()
    q = mln.run(p, precision=precision, snap_every=100, variant="quad", tile=128, steps_per_launch=20)
    ee, ep = _errs(a, q)
    tol = 1e-12 if precision == "fp64" else 1e-5
    assert ee < tol and ep < tol, (ee, ep)


@pytest.mark.parametrize("variant,tile,k,precision", [("quad", 64, 20, "fp64"), ("block", 64, 7, "fp64"),
                                                      ("block", 128, 24, "fp32c"), ("block", 256, 32, "fp32cf"),
                                                      ("wave", 64, 8, "fp64"), ("quad_mfma", 64, 20, "fp32c")])
def test_last_cell_at_a_tile_boundary(orc, variant, tile, k, precision):
    """Grids on which the last cell (whose boundary condition reaches two
    cells back) would be a tile's first owned cell, and its neighbours."""
    for nx in (3 * (tile - 2 * k), 3 * (tile - 2 * k) + 1):
        p = W.random_problem(3, 7, nx=nx, nt=2 * nx + 100)
        ee, ep = _errs(mln.run(p, precision=precision, snap_every=60, variant=variant, tile=tile, steps_per_launch=k),
                       orc.run(p, snap_every=60))
        assert ee < (1e-12 if precision == "fp64" else 1e-5), (nx, ee)


def test_batch_last_cell_at_a_tile_boundary(orc):
    probs = [W.random_problem(2 + i % 2, 80 + i, nx=33 + 16 * i, nt=300) for i in range(4)]
    b = mln.Batch(probs, precision="fp64", snap_every=100, variant="block", tile=64, steps_per_launch=16)
    outs = b.run()
    for p, o in zip(probs, outs):
        ee, ep = _errs({q: v.cpu().numpy() for q, v in o.items()}, orc.run(p, snap_every=100))
        assert ee < 1e-12 and ep < 1e-10, (p.grid.nx, ee, ep)
    b.close()


@pytest.mark.parametrize("variant,tile,k", [("quad", 64, 7), ("block", 64, 7), ("quad", 128, 5)])
def test_adjoint_last_cell_beyond_a_tile(orc, variant, tile, k):
    """Grids on which the last cell would be the first beyond a reverse tile."""
    for nx in (2 * (tile - 2 * k) + k + 1, 2 * (tile - 2 * k) + k):
        p = W.random_problem(3, 7, nx=nx, nt=400)
        gp = 2.0 * p.grid.dt * orc.run(p)["probe"]
        ref = orc.grad(p, gp)
        s = mln.Solver(p, ckpt_every=100)
        s.configure_adjoint(variant, tile, k)
        s.run()
        g = s.grad(gp)
        s.close()
        for q in ref:
            dev = np.max(np.abs(np.asarray(g[q]) - np.asarray(ref[q]))) / np.max(np.abs(ref[q]))
            assert dev < 1e-9, (nx, q, dev)


@pytest.mark.parametrize("nx", [97, 121, 61])
def test_last_cell_and_small_owned_parts(orc, nx):
    """nx - 1 a multiple of many numbers of owned cells, down to two of them."""
    p = W.random_problem(3, 5, nx=nx, nt=200)
    ref = orc.run(p, snap_every=50)
    for variant, tile, k in (("quad", 32, 8), ("quad", 32, 10), ("quad", 32, 15), ("block", 64, 26), ("block", 64, 31)):
        got = mln.run(p, snap_every=50, variant=variant, tile=tile, steps_per_launch=k)
        ee, ep = _errs(got, ref)
        assert ee < 1e-12 and ep < 1e-12, (variant, tile, k, ee, ep)
    b = mln.Batch([p, W.random_problem(3, 6, nx=nx + 1, nt=200)], precision="fp64", snap_every=50, variant="quad",
                  tile=32, steps_per_launch=15)
    ee, ep = _errs({q: v.cpu().numpy() for q, v in b.run()[0].items()}, ref)
    b.close()
    assert ee < 1e-12 and ep < 1e-12, (ee, ep)


@pytest.mark.parametrize("n,variant,precision,tol", [(2, "quad", "fp64", 1e-10), (3, "quad", "fp64", 1e-10),
                                                     (3, "quad_mfma", "fp32c", 1e-5), (3, "quad", "fp32cf", 1e-5),
                                                     (2, "quad", "fp32", 1e-5), (4, "quad", "bf16x6", 1e-4)])
def test_four_lane_boundary_cell(orc, n, variant, precision, tol):
    """The boundary cell, which the lanes of its neighbour keep, at every kind
    of place of a tile: probe, snapshots, and a run in uneven chunks."""
    for nx in list(range(94, 102)) + [3, 34]:
        p = W.random_problem(n, nx, nx=nx, nt=120)
        s = mln.Solver(p, precision=precision, snap_every=40, variant=variant, tile=32, steps_per_launch=8)
        a = {k: v.cpu().numpy().copy() for k, v in s.run().items()}
        s.reset()
        for k in (1, 38, 9):
            s.step(k)
        b = {k: v.cpu().numpy() for k, v in s.run().items()}
        s.close()
        for k in a:
            assert np.array_equal(a[k], b[k]), (nx, k)
        ee, ep = _errs(a, orc.run(p, snap_every=40))
        assert ee < tol and ep < tol, (nx, ee, ep)
