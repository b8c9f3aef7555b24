// tmz.hip -- the two-dimensional TMz solver of include/mln.h (mln_tmz_*):
// validation, factor upload, device state, the per-step launch loop and the
// kernel instantiations of fwd_tmz.hpp.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <memory>
#include <string>
#include <type_traits>
#include <vector>

#include "fwd_tmz_tile.hpp"
#include "handle.hpp"

using namespace mln;

struct mln_tmz {
  Factors f;
  int N = 0, prec = MLN_FP64;
  bool comp = false;
  mln_tmz_grid grid{};
  mln_tmz_record rec{};
  hipStream_t stream = nullptr;
  int64_t nmed = 0, ld = 0, step = 0, nsnap = 0;
  int rs = 8;  // bytes per real
  DevBuf fac, pop, popc;
  FacDev<double> fd{};
  FacDev<float> ff{};
  DevBuf E[2], Hx[2], Hy[2], z[2], src, prof;  // z[1]: the tile kernel only
  int rows = 0, K = 1;  // tile kernel: rows of a tile (0: one step per launch), steps per launch
  int cur = 0, zcur = 0;  // buffers of the current step
  FillPlan fill;
  std::vector<double> src_host, prof_host;
  // FDTD coefficients: chx, chy, ca, cb, 1/dx, 1/dy, kmur (FP64), and the
  // single-precision set with (chx, 1/dx) and (chy, 1/dy) chosen so that
  // their products with cb match the FP64 ones (H_y, H_x carried scaled by
  // chx32/chx and chy32/chy; hs_x, hs_y undo that where H leaves the library)
  double c64[7] = {0, 0, 0, 0, 0, 0, 0};
  float c32[7] = {0, 0, 0, 0, 0, 0, 0};
  double hs_x = 1.0, hs_y = 1.0;
};

namespace {

template <int N, typename Real, bool COMP>
hipError_t launch_n(const TmzArgs<Real> &a, hipStream_t st) {
  const dim3 grid((unsigned)((a.nx + kTmzTX - 1) / kTmzTX), (unsigned)((a.ny + kTmzTY - 1) / kTmzTY));
  if constexpr (N <= 3)
    hipLaunchKernelGGL((fwd_tmz_one_kernel<N, Real, COMP>), grid, dim3(kTmzTX * kTmzTY), 0, st, a);
  else
    hipLaunchKernelGGL((fwd_tmz_kernel<N, Real, COMP>), grid, dim3(kTmzTX * kTmzTY), 0, st, a);
  return hipGetLastError();
}

// rows: C * kTmzWaves
template <int N, typename Real, bool COMP>
hipError_t launch_tile_n(int rows, const TmzTileArgs<Real> &t, hipStream_t st) {
  const dim3 grid((unsigned)((t.a.nx + t.ox - 1) / t.ox), (unsigned)((t.a.ny + t.oy - 1) / t.oy)), block(64 * kTmzWaves);
  switch (rows / kTmzWaves) {
    case 2: hipLaunchKernelGGL((fwd_tmz_tile_kernel<N, Real, COMP, 2, kTmzWaves>), grid, block, 0, st, t); break;
    case 4: hipLaunchKernelGGL((fwd_tmz_tile_kernel<N, Real, COMP, 4, kTmzWaves>), grid, block, 0, st, t); break;
    case 6:
      if constexpr (tmz_six_rows<N, Real, COMP>()) {
        hipLaunchKernelGGL((fwd_tmz_tile_kernel<N, Real, COMP, 6, kTmzWaves>), grid, block, 0, st, t);
        break;
      }
      return hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <typename Real, bool COMP>
hipError_t launch_tile(int N, int rows, const TmzTileArgs<Real> &t, hipStream_t st) {
  return N == 2 ? launch_tile_n<2, Real, COMP>(rows, t, st) : launch_tile_n<3, Real, COMP>(rows, t, st);
}

template <typename Real, bool COMP>
hipError_t launch_tmz(int N, const TmzArgs<Real> &a, hipStream_t st) {
  switch (N) {
    case 2: return launch_n<2, Real, COMP>(a, st);
    case 3: return launch_n<3, Real, COMP>(a, st);
    case 4: return launch_n<4, Real, COMP>(a, st);
    case 6: return launch_n<6, Real, COMP>(a, st);
    default: return hipErrorInvalidValue;
  }
}

// host values -> device reals (FP32: scaled by 1/hscale), into buf at offset 0
template <typename Real>
void to_dev(const double *v, size_t n, double scale, std::vector<unsigned char> &buf) {
  buf.assign(n * sizeof(Real), 0);
  Real *o = (Real *)buf.data();
  for (size_t i = 0; i < n; ++i) o[i] = (Real)(v[i] * scale);
}

template <typename Real>
void from_dev(const std::vector<unsigned char> &buf, size_t n, double scale, double *out) {
  const Real *v = (const Real *)buf.data();
  for (size_t i = 0; i < n; ++i) out[i] = (double)v[i] * scale;
}

int tmz_write_probe0(mln_tmz *t) {
  if (!t->rec.probe_out) return MLN_OK;
  const int64_t nx = t->grid.nx, ny = t->grid.ny;
  std::vector<unsigned char> buf((size_t)nx * ny * t->rs);
  HIP_TRY(hipMemcpy(buf.data(), t->E[t->cur].p, buf.size(), hipMemcpyDeviceToHost));
  std::vector<double> e((size_t)nx * ny), p0(ny);
  if (t->rs == 8)
    from_dev<double>(buf, e.size(), 1.0, e.data());
  else
    from_dev<float>(buf, e.size(), 1.0, e.data());
  for (int64_t j = 0; j < ny; ++j) p0[j] = e[(size_t)j * nx + nx - 1];
  HIP_TRY(hipMemcpy(t->rec.probe_out, p0.data(), ny * sizeof(double), hipMemcpyHostToDevice));
  return MLN_OK;
}

int tmz_reset(mln_tmz *t) {
  HIP_TRY(t->fill.run(t->stream));
  t->cur = t->zcur = 0;
  t->step = 0;
  HIP_TRY(hipStreamSynchronize(t->stream));
  return MLN_OK;
}

// The plan of the state at step 0: the source column, zero fields, the
// rotation route's initial deviation y0 in every medium cell (then its low
// parts with the compensated state); the probe's first row (column nx - 1,
// nx >= 3) is zero.
int tmz_plan(mln_tmz *t) {
  const int64_t nx = t->grid.nx, ny = t->grid.ny;
  std::vector<double> e0(t->prof_host), z0(t->f.y0);
  for (double &v : e0) v *= t->src_host[0];
  if (t->comp)
    for (int k = 0; k < t->f.D; ++k) z0.push_back(z0[k] - (double)(float)z0[k]);
  for (int b = 0; b < 2; ++b) {
    t->fill.add(t->E[b].p, ny, nx, 1, e0, t->rs);
    t->fill.add(t->Hx[b].p, ny, nx, 0, {}, t->rs);
    t->fill.add(t->Hy[b].p, ny, nx, 0, {}, t->rs);
  }
  t->fill.add(t->z[0].p, (int64_t)z0.size(), t->ld, t->nmed, z0, t->rs);
  t->fill.add(t->rec.probe_out, 1, ny, 0, {}, 8);
  return t->fill.upload();
}

template <typename Real>
TmzArgs<Real> tmz_args(mln_tmz *t, const FacDev<Real> &fd, const Real (&c)[7]) {
  TmzArgs<Real> a{};
  a.fac = fd;
  const int in = t->cur, out = 1 - t->cur;
  a.Ein = (const Real *)t->E[in].p;
  a.Eout = (Real *)t->E[out].p;
  a.Hxin = (const Real *)t->Hx[in].p;
  a.Hxout = (Real *)t->Hx[out].p;
  a.Hyin = (const Real *)t->Hy[in].p;
  a.Hyout = (Real *)t->Hy[out].p;
  a.z = (Real *)t->z[t->zcur].p;
  a.src = (const Real *)t->src.p;
  a.prof = (const Real *)t->prof.p;
  a.nx = t->grid.nx;
  a.ny = t->grid.ny;
  a.mx0 = t->grid.mx0;
  a.mx1 = t->grid.mx1;
  a.my0 = t->grid.my0;
  a.my1 = t->grid.my1;
  if (t->nmed == 0) a.mx0 = a.mx1 = 0x7fffff00;  // no tile crosses a medium of no cells
  a.ld = t->ld;
  a.chx = c[0];
  a.chy = c[1];
  a.ca = c[2];
  a.cb = c[3];
  a.idx = c[4];
  a.idy = c[5];
  a.kmur = c[6];
  a.pop_out = t->rec.pop_out;
  a.e_out = t->rec.e_out;
  a.probe_out = t->rec.probe_out;
  a.opaque0 = 0;
  return a;
}

// Rows of the tiles of a launch of K >= 2 steps and, in *us, its time: the
// least in a model of a launch, 2.5 us plus the larger of a tile's own time
// (its loads and stores and K steps) times the tiles that a compute unit works
// off one after the other, and of the whole grid's memory traffic (4.6 TB/s)
// and arithmetic one after the other (the workgroup that fills a compute
// unit's registers loads, steps and stores in turn).  Fitted to beams of 150 x
// 30 and 2048 x 512 cells, us per launch model / measured on the larger:
// three-level FP64 48 rows and 5 steps 79 / 78, 6 steps 99 / 91, 3 steps 60 /
// 59, 32 rows and 5 steps 87 / 85, 16 rows and 3 steps 58 / 51; FP32 32 rows
// and 6 steps 63 / 59.
int tmz_rows(const mln_tmz *t, int K, double *us) {
  // [N = 2, 3][FP64, FP32][16, 32, 48 rows]: us of the ends of a tile and of a
  // step of it, and tiles that share a compute unit
  static const double ends[2][2][3] = {{{1.6, 2.6, 0}, {1.2, 1.9, 0}}, {{2.5, 5.4, 6.4}, {1.8, 3.2, 0}}};
  static const double step[2][2][3] = {{{1.2, 2.0, 0}, {0.95, 1.5, 0}}, {{2.07, 3.63, 5.78}, {1.55, 2.85, 0}}};
  static const double share[2][2][3] = {{{1.7, 1.6, 0}, {1.8, 1.9, 0}}, {{1.5, 1.0, 1.0}, {1.8, 1.4, 0}}};
  // arithmetic of a medium cell and step, us per cell of the grid
  static const double cell[2][2] = {{1.0e-6, 0.85e-6}, {4.8e-6, 3.2e-6}};
  const mln_tmz_grid &g = t->grid;
  const int ni = t->N == 2 ? 0 : 1, pi = t->prec == MLN_FP32 ? 1 : 0, cus = device_cus();
  const double all = (double)g.nx * (double)g.ny, med = t->nmed / all;
  const double bytes = t->rs * (3.0 + med * (t->comp ? 2 : 1) * t->f.D);
  double best = 0.0;
  int best_rows = 0;
  for (int c = 0; c < 3; ++c) {
    const int rows = 16 * (c + 1);
    if (step[ni][pi][c] == 0 || 3 * K > rows + 2) continue;
    const int64_t ox = kTmzTileX - 2 * K, oy = rows - 2 * K;
    const double tiles = (double)((g.nx + ox - 1) / ox) * (double)((g.ny + oy - 1) / oy);
    const double cells = tiles * rows * kTmzTileX, n = tiles / (cus * share[ni][pi][c]);
    const double own = std::max(1.0, n) * (ends[ni][pi][c] + K * step[ni][pi][c]);
    // (two workgroups share a compute unit at 16 rows: half of the arithmetic overlaps)
    const double arith = cells * K * (0.15 + 0.85 * med) * cell[ni][pi] * (c == 0 ? 0.45 : 1.0);
    const double x = 2.5 + std::max(own, (cells + all) * bytes / 4.6e6 + arith);
    if (best_rows == 0 || x < best) {
      best = x;
      best_rows = rows;
    }
  }
  if (us) *us = best;
  return best_rows;
}

// Steps per launch: the least time per step.  Against one step per launch, us
// per step on the beam of 2048 x 512 cells: three-level FP64 15.6 / 27.1,
// compensated FP32 17.8 / 25.0, FP32 10.0 / 15.6.
void tmz_shape(mln_tmz *t) {
  if (t->N > 3 || t->grid.nx > (int64_t)1 << 30) return;  // one step per launch
  double best = 0.0;
  for (int K = 2; K <= 11; ++K) {
    double us = 0.0;
    const int rows = tmz_rows(t, K, &us);
    if (rows && (best == 0.0 || us / K < best)) {
      best = us / K;
      t->rows = rows;
      t->K = K;
    }
  }
}

// Columns a tile owns in a launch of k steps.  The Mur column needs the new E
// of its left neighbour, one cell deeper into the halo: it must not be a
// tile's first column.
int tmz_columns(int64_t nx, int k) {
  int ox = kTmzTileX - 2 * k;
  while ((nx - 1) % ox == 0 && ox > 1) --ox;
  return ox;
}

template <typename Real>
int tmz_steps_typed(mln_tmz *t, const FacDev<Real> &fd, const Real (&c)[7], int64_t n) {
  const int64_t se = t->rec.snap_every;
  for (int64_t s = 0; s < n;) {
    TmzArgs<Real> a = tmz_args<Real>(t, fd, c);
    a.n = t->step;
    const int k = (int)std::min<int64_t>(t->K, n - s);
    hipError_t e;
    if (k > 1) {
      const int rows = k == t->K ? t->rows : tmz_rows(t, k, nullptr);
      TmzTileArgs<Real> q{};
      q.a = a;
      q.zout = (Real *)t->z[1 - t->zcur].p;
      q.nsteps = k;
      q.halo = k;
      q.ox = tmz_columns(t->grid.nx, k);
      q.oy = rows - 2 * k;
      q.s_snap = -1;
      if (se > 0) {  // the first step of the launch that completes a snapshot
        q.a.snap_i = t->step / se;
        const int64_t f = (q.a.snap_i + 1) * se - 1 - t->step;
        if (f < k) q.s_snap = (int)f;
        q.gap = (int)std::min<int64_t>(se, kTmzTileMaxSteps);
      }
      if constexpr (sizeof(Real) == 8)
        e = launch_tile<double, false>(t->N, rows, q, t->stream);
      else
        e = t->comp ? launch_tile<float, true>(t->N, rows, q, t->stream)
                    : launch_tile<float, false>(t->N, rows, q, t->stream);
      t->zcur = 1 - t->zcur;
    } else {
      a.snap = (se > 0 && (t->step + 1) % se == 0) ? 1 : 0;
      a.snap_i = se > 0 ? (t->step + 1) / se - 1 : 0;
      if constexpr (sizeof(Real) == 8)
        e = launch_tmz<double, false>(t->N, a, t->stream);
      else
        e = t->comp ? launch_tmz<float, true>(t->N, a, t->stream) : launch_tmz<float, false>(t->N, a, t->stream);
    }
    if (e != hipSuccess) return set_err(MLN_EHIP, std::string("TMz launch: ") + hipGetErrorString(e));
    t->cur = 1 - t->cur;
    t->step += k;
    s += k;
  }
  return MLN_OK;
}

int tmz_steps(mln_tmz *t, int64_t n) {
  if (t->rs == 8) {
    const double(&c)[7] = t->c64;
    return tmz_steps_typed<double>(t, t->fd, c, n);
  }
  const float(&c)[7] = t->c32;
  return tmz_steps_typed<float>(t, t->ff, c, n);
}

}  // namespace

extern "C" {

int mln_tmz_init(const mln_medium *medium, const mln_tmz_grid *grid, const mln_tmz_source *source,
                 const mln_tmz_record *record, int32_t precision, void *stream, mln_tmz **out) {
  if (!out) return set_err(MLN_EINVAL, "null output handle");
  *out = nullptr;
  if (!medium || !grid || !source) return set_err(MLN_EINVAL, "need a medium, a grid and a source");
  const mln_tmz_grid &g = *grid;
  if (g.nx < 3 || g.ny < 1 || g.nt < 0) return set_err(MLN_EINVAL, "need nx >= 3, ny >= 1, nt >= 0");
  if (g.ny > (int64_t)kTmzTY * 65535) return set_err(MLN_EINVAL, "ny beyond the launch grid");
  if (!(g.dx > 0) || !(g.dy > 0) || !(g.dt > 0) || !std::isfinite(g.dx) || !std::isfinite(g.dy) ||
      !std::isfinite(g.dt))
    return set_err(MLN_EINVAL, "dx, dy and dt must be positive");
  if (g.mx0 < 1 || g.mx1 < g.mx0 || g.mx1 > g.nx - 1 || g.my0 < 0 || g.my1 < g.my0 || g.my1 > g.ny)
    return set_err(MLN_EINVAL, "medium must satisfy 1 <= mx0 <= mx1 <= nx-1 and 0 <= my0 <= my1 <= ny");
  if (!(g.eps_r > 0) || !(g.mu_r > 0) || !(g.sigma >= 0))
    return set_err(MLN_EINVAL, "eps_r, mu_r must be > 0 and sigma >= 0");
  if (!source->samples || source->n < g.nt + 1 || !source->profile || !std::isfinite(source->amplitude))
    return set_err(MLN_EINVAL, "source needs nt + 1 samples, a finite amplitude and a profile");
  for (int64_t n = 0; n <= g.nt; ++n)
    if (!std::isfinite(source->samples[n])) return set_err(MLN_EINVAL, "non-finite source sample");
  for (int64_t j = 0; j < g.ny; ++j)
    if (!std::isfinite(source->profile[j])) return set_err(MLN_EINVAL, "non-finite source profile");
  if (precision != MLN_FP64 && precision != MLN_FP32 && precision != MLN_FP32_COMP)
    return set_err(MLN_ENOTSUPPORTED, "the TMz solver is built for MLN_FP64, MLN_FP32 and MLN_FP32_COMP");
  const double eps = kEps0 * g.eps_r, mu = kMu0 * g.mu_r;
  const double cl = 1.0 / std::sqrt(eps * mu);
  if (cl * g.dt * std::sqrt(1.0 / (g.dx * g.dx) + 1.0 / (g.dy * g.dy)) > 1.0)
    return set_err(MLN_ECOURANT, "2-D Yee update unstable: c dt sqrt(1/dx^2 + 1/dy^2) > 1");

  std::unique_ptr<mln_tmz> t(new mln_tmz());
  std::string err;
  int rc = build_factors(medium, g.dt, &t->f, &err);
  if (rc) return set_err(rc, err);
  t->N = t->f.N;
  if (t->N != 2 && t->N != 3 && t->N != 4 && t->N != 6)
    return set_err(MLN_ENOTSUPPORTED, "the TMz kernels are built for N = 2, 3, 4 and 6");
  t->grid = g;
  t->rec = record ? *record : mln_tmz_record{};
  if (t->rec.snap_every < 0) return set_err(MLN_EINVAL, "snap_every must be >= 0");
  t->nsnap = t->rec.snap_every > 0 ? g.nt / t->rec.snap_every : 0;
  if (t->nsnap == 0) {
    t->rec.e_out = nullptr;
    t->rec.pop_out = nullptr;
  }
  t->prec = precision;
  t->comp = precision == MLN_FP32_COMP;
  t->rs = precision == MLN_FP64 ? 8 : 4;
  t->stream = (hipStream_t)stream;
  t->nmed = (g.mx1 - g.mx0) * (g.my1 - g.my0);
  t->ld = std::max<int64_t>(1, (t->nmed + 63) / 64 * 64);
  // FDTD coefficients (2-D form of Eq. maxwell, semi-implicit sigma)
  const double sg = g.sigma * g.dt / (2.0 * eps);
  t->c64[0] = g.dt / (mu * g.dx);
  t->c64[1] = g.dt / (mu * g.dy);
  t->c64[2] = (1.0 - sg) / (1.0 + sg);
  t->c64[3] = (g.dt / eps) / (1.0 + sg);
  t->c64[4] = 1.0 / g.dx;
  t->c64[5] = 1.0 / g.dy;
  t->c64[6] = (cl * g.dt - g.dx) / (cl * g.dt + g.dx);
  for (int k = 0; k < 7; ++k) t->c32[k] = (float)t->c64[k];
  courant_pair32(t->c64[0], t->c64[3], t->c64[4], t->c32[0], t->c32[4]);
  courant_pair32(t->c64[1], t->c64[3], t->c64[5], t->c32[1], t->c32[5]);
  t->hs_x = t->c64[1] / (double)t->c32[1];  // H_x is carried scaled by chy32 / chy
  t->hs_y = t->c64[0] / (double)t->c32[0];  // H_y by chx32 / chx
  if (t->rs == 8) {
    rc = upload_factors<double>(t->f, MLN_ROUTE_ROTATION, g.dt, t->fac, t->pop, t->popc, t->fd);
  } else {
    rc = upload_factors<float>(t->f, MLN_ROUTE_ROTATION, g.dt, t->fac, t->pop, t->popc, t->ff);
  }
  if (rc) return rc;
  // source samples (amplitude applied) and profile in the field precision
  t->src_host.resize(g.nt + 1);
  for (int64_t n = 0; n <= g.nt; ++n) t->src_host[n] = source->amplitude * source->samples[n];
  t->prof_host.assign(source->profile, source->profile + g.ny);
  std::vector<unsigned char> buf;
  const size_t cells = (size_t)g.nx * g.ny;
  if (t->rs == 8) to_dev<double>(t->src_host.data(), t->src_host.size(), 1.0, buf);
  else to_dev<float>(t->src_host.data(), t->src_host.size(), 1.0, buf);
  HIP_TRY(t->src.alloc(buf.size()));
  HIP_TRY(hipMemcpy(t->src.p, buf.data(), buf.size(), hipMemcpyHostToDevice));
  if (t->rs == 8) to_dev<double>(t->prof_host.data(), g.ny, 1.0, buf);
  else to_dev<float>(t->prof_host.data(), g.ny, 1.0, buf);
  HIP_TRY(t->prof.alloc(buf.size()));
  HIP_TRY(hipMemcpy(t->prof.p, buf.data(), buf.size(), hipMemcpyHostToDevice));
  for (int b = 0; b < 2; ++b) {
    HIP_TRY(t->E[b].alloc(cells * t->rs));
    HIP_TRY(t->Hx[b].alloc(cells * t->rs));
    HIP_TRY(t->Hy[b].alloc(cells * t->rs));
  }
  const int D = t->f.D;
  tmz_shape(t.get());
  const size_t zb = (size_t)(t->comp ? 2 * D : D) * t->ld * t->rs;
  HIP_TRY(t->z[0].alloc(zb));
  if (t->rows) {
    size_t free_bytes = 0, total = 0;
    HIP_TRY(hipMemGetInfo(&free_bytes, &total));
    hipError_t e = hipErrorOutOfMemory;
    if (second_buffer_fits(zb, free_bytes)) e = t->z[1].alloc(zb);
    if (e == hipErrorOutOfMemory) {  // no room for a second state: one step per launch, in place
      (void)hipGetLastError();
      t->z[1].p = nullptr;
      t->rows = 0;
      t->K = 1;
    } else {
      HIP_TRY(e);
    }
  }
  rc = tmz_plan(t.get());
  if (rc) return rc;
  rc = tmz_reset(t.get());
  if (rc) return rc;
  *out = t.release();
  return MLN_OK;
}

int mln_tmz_step(mln_tmz *t, int64_t n_steps) {
  if (!t) return set_err(MLN_EINVAL, "null handle");
  if (n_steps < 0) return set_err(MLN_EINVAL, "n_steps must be >= 0");
  return tmz_steps(t, std::min<int64_t>(n_steps, t->grid.nt - t->step));
}

int mln_tmz_run(mln_tmz *t) {
  if (!t) return set_err(MLN_EINVAL, "null handle");
  const int rc = mln_tmz_step(t, t->grid.nt - t->step);
  if (rc) return rc;
  HIP_TRY(hipStreamSynchronize(t->stream));
  return MLN_OK;
}

int mln_tmz_reset(mln_tmz *t) {
  if (!t) return set_err(MLN_EINVAL, "null handle");
  return tmz_reset(t);
}

int mln_tmz_current_step(const mln_tmz *t, int64_t *step) {
  if (!t || !step) return set_err(MLN_EINVAL, "null argument");
  *step = t->step;
  return MLN_OK;
}

int mln_tmz_set_fields(mln_tmz *t, const double *Ez, const double *Hx, const double *Hy) {
  if (!t) return set_err(MLN_EINVAL, "null handle");
  const size_t cells = (size_t)t->grid.nx * t->grid.ny;
  for (const double *a : {Ez, Hx, Hy})
    for (size_t i = 0; a && i < cells; ++i)
      if (!std::isfinite(a[i])) return set_err(MLN_EINVAL, "non-finite field value");
  HIP_TRY(hipStreamSynchronize(t->stream));
  std::vector<unsigned char> buf;
  const double sx = t->rs == 8 ? 1.0 : 1.0 / t->hs_x, sy = t->rs == 8 ? 1.0 : 1.0 / t->hs_y;
  const double *src[3] = {Ez, Hx, Hy};
  const double scale[3] = {1.0, sx, sy};
  DevBuf *dst[3] = {&t->E[t->cur], &t->Hx[t->cur], &t->Hy[t->cur]};
  for (int k = 0; k < 3; ++k) {
    if (!src[k]) continue;
    if (t->rs == 8) to_dev<double>(src[k], cells, scale[k], buf);
    else to_dev<float>(src[k], cells, scale[k], buf);
    HIP_TRY(hipMemcpy(dst[k]->p, buf.data(), buf.size(), hipMemcpyHostToDevice));
  }
  if (Ez && t->step == 0) return tmz_write_probe0(t);
  return MLN_OK;
}

int mln_tmz_get_fields(mln_tmz *t, double *Ez, double *Hx, double *Hy) {
  if (!t) return set_err(MLN_EINVAL, "null handle");
  const size_t cells = (size_t)t->grid.nx * t->grid.ny;
  HIP_TRY(hipStreamSynchronize(t->stream));
  std::vector<unsigned char> buf(cells * t->rs);
  double *dst[3] = {Ez, Hx, Hy};
  const double scale[3] = {1.0, t->rs == 8 ? 1.0 : t->hs_x, t->rs == 8 ? 1.0 : t->hs_y};
  DevBuf *src[3] = {&t->E[t->cur], &t->Hx[t->cur], &t->Hy[t->cur]};
  for (int k = 0; k < 3; ++k) {
    if (!dst[k]) continue;
    HIP_TRY(hipMemcpy(buf.data(), src[k]->p, buf.size(), hipMemcpyDeviceToHost));
    if (t->rs == 8) from_dev<double>(buf, cells, scale[k], dst[k]);
    else from_dev<float>(buf, cells, scale[k], dst[k]);
  }
  return MLN_OK;
}

void mln_tmz_free(mln_tmz *t) {
  if (!t) return;
  (void)hipStreamSynchronize(t->stream);
  delete t;
}

}  // extern "C"
