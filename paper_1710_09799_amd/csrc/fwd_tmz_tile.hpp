// fwd_tmz_tile.hpp -- several time steps of the 2-D TMz grid per launch, N = 2,
// 3 (the step itself: fwd_tmz.hpp, cells.hpp).
//
// One step per launch reads and writes every field and the whole Bloch state
// once per step (three-level FP64: 176 B per medium cell), which bounds it by
// memory.  Here a workgroup holds a tile of 64 columns x C NW rows in
// registers for nsteps <= halo steps and writes back its inner part: the error
// made at the tile's edges travels inwards by one cell per step.
//   * lane l of wavefront w carries the C cells of column l in rows w C ..
//     w C + C - 1: the neighbours in y are the lane's own registers, those in
//     x a wavefront shift (DPP);
//   * between wavefronts only the first and the last row of E pass through
//     LDS, written before the medium step and read after the one barrier of a
//     step (two buffers); the H_x face below a wavefront's first row is a
//     private copy, updated with its owner's operands;
//   * the medium step takes the cells of a lane together (cells.hpp);
//     wavefronts whose cells are all medium, or none, take no per-cell test.
// The Bloch state has two buffers, as the fields do: a tile's halo reads the
// old state of cells that other tiles write.  Rows wrap (periodic in y), also
// more than once where ny is smaller than the tile.
//
// Measured, three-level beam of 2048 x 512 cells, us per step, one step per
// launch with a cell per thread / this kernel with the shape the host takes:
// FP64 27.1 / 16.3, FP32 15.6 / 9.7, compensated FP32 25.0 / 18.4.  The
// workgroup's registers leave one or two of them per compute unit, so its loads
// (a third of the launch) are not hidden behind another's arithmetic.
#pragma once

#include "cells.hpp"
#include "fwd_tmz.hpp"
#include "fwd_wave.hpp"

namespace mln {

constexpr int kTmzTileX = 64;         // columns of a tile (one wavefront)
constexpr int kTmzTileMaxSteps = 16;  // steps per launch
constexpr int kTmzWaves = 8;          // wavefronts of a tile

template <typename Real>
struct TmzTileArgs {
  TmzArgs<Real> a;   // a.z: the state before the launch, a.n: its first step
  Real *zout;
  int nsteps, halo;  // steps of this launch <= halo
  int ox, oy;        // columns and rows a tile owns
  int s_snap, gap;   // first recording step of the launch (-1: none), steps between recordings
};

// The argument block in constant memory: what only a recording step, an edge
// tile or the ends of the launch need is read from it again (as in
// fwd_lane.hpp), not held in scalar registers through the step loop.
template <typename Real>
using TmzCold = const __attribute__((address_space(4))) TmzTileArgs<Real> *;
template <typename Real>
__device__ __forceinline__ TmzCold<Real> tmz_again(TmzCold<Real> p) {
  __asm__ volatile("" : "+s"(p));
  return p;
}

// The instance of six rows per lane: what fits 256 registers only in FP64
// (N = 3); FP32 tiles gain nothing from it.
template <int N, typename Real, bool COMP>
constexpr bool tmz_six_rows() {
  return N == 3 && (COMP || sizeof(Real) == 8);
}

// Cells stepped together: their temporaries live beside all C states.
template <int N, typename M, int C>
constexpr int tmz_group() {
  return N == 2 ? (C < 4 ? C : 4) : (sizeof(M) == 8 ? (C < 2 ? C : 2) : (C < 4 ? C : 4));
}

template <int N, typename Real, bool COMP, int C, int NW>
__global__ void __launch_bounds__(64 * NW) fwd_tmz_tile_kernel(TmzTileArgs<Real> t) {
  typedef typename CellType<Real, COMP>::type M;
  constexpr int D = N * N - 1;
  constexpr int G = tmz_group<N, M, C>();
  static_assert(C % G == 0, "whole groups");
  __shared__ Real sLo[2][NW][64], sHi[2][NW][64];
  __shared__ Real sSrc[kTmzTileMaxSteps];
  const TmzArgs<Real> &a = t.a;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int nx = (int)a.nx, ny = (int)a.ny;  // the host takes this kernel only where cells fit 31 bits
  const int x0 = (int)blockIdx.x * t.ox - t.halo, i = x0 + lane;
  const int y0 = (int)blockIdx.y * t.oy - t.halo + w * C;  // first row of the wavefront, unwrapped
  const int mx0 = (int)a.mx0, mx1 = (int)a.mx1, my0 = (int)a.my0, my1 = (int)a.my1;
  const int64_t mw = mx1 - mx0;
  const TmzCold<Real> cold = (TmzCold<Real>)__builtin_amdgcn_kernarg_segment_ptr();
  auto wrap = [&](int j) {
    j %= ny;
    return j < 0 ? j + ny : j;
  };
  CellFac<N, M> F;
  F.set(a.fac);
  CellK<N, M> K;
  K.load(F);

  const bool in_x = i >= 0 && i < nx;
  const bool col_med = i >= mx0 && i < mx1;
  const bool cols_any = x0 < mx1 && x0 + 64 > mx0, cols_all = x0 >= mx0 && x0 + 64 <= mx1;
  Real E[C], Hx[C], Hy[C], Hxd = 0;
  M z[C][D];
  int row_med = 0;  // bit c: row c crosses the medium (uniform)
  // every load unconditional, from the nearest cell of the grid or of the
  // medium where the lane's own is outside, so that all are in flight at once
  const int ic = i < 0 ? 0 : (i < nx ? i : nx - 1);
  const int im = i < mx0 ? 0 : (i < mx1 ? i - mx0 : (mx1 > mx0 ? mx1 - mx0 - 1 : 0));
  Real zl[C][COMP ? D : 1];
  Real zh[C][D];
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int j = wrap(y0 + c);
    const int64_t g = (int64_t)j * nx + ic;
    E[c] = a.Ein[g];
    Hx[c] = a.Hxin[g];
    Hy[c] = a.Hyin[g];
    const bool rm = j >= my0 && j < my1;
    row_med |= (int)rm << c;
    if (cols_any && rm) {
      const int64_t m = (int64_t)(j - my0) * mw + im;
#pragma unroll
      for (int k = 0; k < D; ++k) {
        zh[c][k] = a.z[k * a.ld + m];
        if constexpr (COMP) zl[c][k] = a.z[(D + k) * a.ld + m];
      }
    } else {
#pragma unroll
      for (int k = 0; k < D; ++k) {
        zh[c][k] = 0;
        if constexpr (COMP) zl[c][k] = 0;
      }
    }
  }
  Hxd = a.Hxin[(int64_t)wrap(y0 - 1) * nx + ic];
#pragma unroll
  for (int c = 0; c < C; ++c) {
    E[c] = in_x ? E[c] : Real(0);
#pragma unroll
    for (int k = 0; k < D; ++k) {
      M v = (M)zh[c][k];
      if constexpr (COMP) v += (M)zl[c][k];
      z[c][k] = col_med ? v : M(0);
    }
  }
  const bool any_med = cols_any && row_med;
  const bool all_med = cols_all && row_med == (1 << C) - 1;
  const bool inside = x0 >= 1 && x0 + 64 <= nx - 1;  // no source or boundary column, none beyond the grid
  if (threadIdx.x < (unsigned)t.nsteps) sSrc[threadIdx.x] = a.src[a.n + 1 + threadIdx.x];
  // whether this tile writes row c of this lane's column
  auto owned = [&](TmzCold<Real> q, int c) {
    const int lx = lane - q->halo, r = w * C + c - q->halo;
    return lx >= 0 && lx < q->ox && i < (int)q->a.nx && r >= 0 && r < q->oy &&
           (int)blockIdx.y * q->oy + r < (int)q->a.ny;
  };
  int s_snap = t.s_snap, snaps = 0;
  __syncthreads();

  for (int s = 0; s < t.nsteps; ++s) {
    const bool snap = s == s_snap;
    const int b = s & 1;
    sLo[b][w][lane] = E[0];
    sHi[b][w][lane] = E[C - 1];
    M P[C];
#pragma unroll
    for (int c = 0; c < C; ++c) P[c] = 0;
    if (any_med) {
#pragma unroll
      for (int q = 0; q < C; q += G) {
        M e[G], p[G], y[G][D];
#pragma unroll
        for (int c = 0; c < G; ++c) {
          e[c] = (M)E[q + c];
#pragma unroll
          for (int k = 0; k < D; ++k) y[c][k] = z[q + c][k];
        }
        // (six rows per lane fill the registers and spill around calls)
        cells_rotate<N, M, G, C == 6 ? Wide::inlined : Wide::calls>(F, e, y);
        if (__builtin_expect(snap, 0)) {
          const TmzCold<Real> cq = tmz_again<Real>(cold);
          double *pop = cq->a.pop_out;
          const int rows = (int)cq->a.my1 - (int)cq->a.my0, cols = (int)cq->a.mx1 - (int)cq->a.mx0;
          const int64_t nm = (int64_t)rows * cols;
          if (pop) {
#pragma unroll
            for (int c = 0; c < G; ++c)
              if (((row_med >> (q + c)) & 1) && col_med && owned(cq, q + c)) {
                const int64_t m = (int64_t)(wrap(y0 + q + c) - (int)cq->a.my0) * cols + (i - (int)cq->a.mx0);
                cells_record<N, M>(cq->a.fac.pop, cq->a.fac.popc, y[c], pop + (cq->a.snap_i + snaps) * N * nm + m, nm);
              }
          }
        }
        cells_shared<N, M, COMP, G>(F, K, y, p);
#pragma unroll
        for (int c = 0; c < G; ++c) {
          P[q + c] = p[c];
#pragma unroll
          for (int k = 0; k < D; ++k) z[q + c][k] = y[c][k];
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if (!all_med) {  // cells beside the medium keep no state and no polarisation
#pragma unroll
        for (int c = 0; c < C; ++c) {
          int med = col_med && ((row_med >> c) & 1);
          __asm__ volatile("" : "+v"(med));  // keeps the selects inside this branch
          P[c] = med ? P[c] : M(0);
#pragma unroll
          for (int k = 0; k < D; ++k) z[c][k] = med ? z[c][k] : M(0);
        }
      }
    }
    lds_barrier();
    const Real Eup = w + 1 < NW ? sLo[b][w + 1 < NW ? w + 1 : 0][lane] : Real(0);
    const Real Edn = w > 0 ? sHi[b][w > 0 ? w - 1 : 0][lane] : Real(0);
    // H^{n+1/2}, then E^{n+1} row by row upwards (row c + 1 still holds E^n
    // when row c needs it); faces outside the grid are updated too, nothing
    // reads them
    Hxd = tmz_hx(Hxd, a.chy, E[0], Edn);
    Real below = Hxd;
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const Real up = c + 1 < C ? E[c + 1 < C ? c + 1 : 0] : Eup;
      Hx[c] = tmz_hx(Hx[c], a.chy, up, E[c]);
      const Real Er = wave_shift<kDppWaveShl1>(E[c]);
      Hy[c] = tmz_hy(Hy[c], a.chx, Er, E[c]);
      const Real hyl = wave_shift<kDppWaveShr1>(Hy[c]);
      const Real curl = (Hy[c] - hyl) * a.idx - (Hx[c] - below) * a.idy;
      const Real En = a.ca * E[c] + a.cb * (-(Real)P[c] + curl);
      below = Hx[c];
      if (inside) {
        E[c] = En;
      } else {
        const Real El = wave_shift<kDppWaveShr1>(E[c]);
        const Real Enl = wave_shift<kDppWaveShr1>(En);
        const TmzCold<Real> cq = tmz_again<Real>(cold);
        const int j = wrap(y0 + c), last = (int)cq->a.nx - 1;
        Real v = (i >= 1 && i < last) ? En : E[c];
        if (i == 0) v = sSrc[s] * cq->a.prof[j];
        if (i == last) {  // first-order Mur boundary (column nx-2 >= 1 is interior)
          v = El + cq->a.kmur * (Enl - E[c]);
          if (cq->a.probe_out && owned(cq, c)) cq->a.probe_out[(cq->a.n + s + 1) * cq->a.ny + j] = (double)v;
        }
        E[c] = v;
      }
    }
    if (__builtin_expect(snap, 0)) {
      const TmzCold<Real> cq = tmz_again<Real>(cold);
      if (cq->a.e_out) {
        double *e = cq->a.e_out + (cq->a.snap_i + snaps) * cq->a.nx * cq->a.ny + i;
#pragma unroll
        for (int c = 0; c < C; ++c)
          if (owned(cq, c)) e[(int64_t)wrap(y0 + c) * cq->a.nx] = (double)E[c];
      }
      s_snap += cq->gap;
      ++snaps;
    }
  }
  const TmzCold<Real> cq = tmz_again<Real>(cold);
  const int64_t ld = cq->a.ld;
  Real *zout = cq->zout;
#pragma unroll
  for (int c = 0; c < C; ++c) {
    if (!owned(cq, c)) continue;
    const int j = wrap(y0 + c);
    const int64_t g = (int64_t)j * cq->a.nx + i;
    cq->a.Eout[g] = E[c];
    cq->a.Hxout[g] = Hx[c];
    if (i <= (int)cq->a.nx - 2) cq->a.Hyout[g] = Hy[c];
    if (col_med && ((row_med >> c) & 1)) {
      const int64_t m = (int64_t)(j - (int)cq->a.my0) * (cq->a.mx1 - cq->a.mx0) + (i - (int)cq->a.mx0);
#pragma unroll
      for (int k = 0; k < D; ++k) {
        const Real hi = (Real)z[c][k];
        zout[k * ld + m] = hi;
        if constexpr (COMP) zout[(D + k) * ld + m] = (Real)(z[c][k] - (M)hi);
      }
    }
  }
}

// One step per launch of the same arithmetic, the Bloch state in place: a
// cell per lane, one row of 64 columns per wavefront.  Launches of one step
// take it (memory bound, and small workgroups overlap loads and arithmetic
// where one that fills a compute unit can not: three-level FP64, 2048 x 512
// cells, 22.8 us per step against 32 to 39 with the tiles above), and
// whole runs on grids with no room for a second Bloch state or beyond the
// tiles' 32-bit cell indices.
template <int N, typename Real, bool COMP>
__global__ void __launch_bounds__(kTmzTX * kTmzTY) fwd_tmz_one_kernel(TmzArgs<Real> a) {
  typedef typename CellType<Real, COMP>::type M;
  constexpr int D = N * N - 1;
  const int64_t nx = a.nx, ny = a.ny;
  const int64_t x0 = (int64_t)blockIdx.x * kTmzTX, i = x0 + (threadIdx.x & 63);
  const int64_t j = (int64_t)blockIdx.y * kTmzTY + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  if (j >= ny) return;  // whole wavefronts
  const int64_t ic = i < nx ? i : nx - 1, il = ic > 0 ? ic - 1 : 0, ir = ic + 1 < nx ? ic + 1 : ic;
  const Real *row = a.Ein + j * nx, *hxr = a.Hxin + j * nx, *hyr = a.Hyin + j * nx;
  const int64_t jp = j + 1 == ny ? 0 : j + 1, jm = j == 0 ? ny - 1 : j - 1;
  const bool med = i >= a.mx0 && i < a.mx1, rm = j >= a.my0 && j < a.my1;
  const bool any = rm && x0 < a.mx1 && x0 + 64 > a.mx0;
  const int64_t mw = a.mx1 - a.mx0, nmed = mw * (a.my1 - a.my0);
  const int64_t im = i < a.mx0 ? 0 : (i < a.mx1 ? i - a.mx0 : (mw > 0 ? mw - 1 : 0)), m = (j - a.my0) * mw + im;
  Real zh[D], zl[COMP ? D : 1];
  if (any) {
#pragma unroll
    for (int k = 0; k < D; ++k) {
      zh[k] = a.z[k * a.ld + m];
      if constexpr (COMP) zl[k] = a.z[(D + k) * a.ld + m];
    }
  }
  const Real E = row[ic], El = row[il], Er = row[ir], Eup = a.Ein[jp * nx + ic], Edn = a.Ein[jm * nx + ic];
  const Real hx0 = hxr[ic], hxd0 = a.Hxin[jm * nx + ic], hy0 = hyr[ic], hyl0 = hyr[il];
  M P[1] = {0};
  if (any) {
    CellFac<N, M> F;
    F.set(a.fac);
    CellK<N, M> K;
    K.load(F);
    M e[1] = {(M)E}, z[1][D];
#pragma unroll
    for (int k = 0; k < D; ++k) {
      z[0][k] = (M)zh[k];
      if constexpr (COMP) z[0][k] += (M)zl[k];
    }
    cells_rotate<N, M, 1, sizeof(M) == 8 ? Wide::inlined : Wide::calls>(F, e, z);
    if (a.snap && a.pop_out && med) cells_record<N, M>(a.fac.pop, a.fac.popc, z[0], a.pop_out + a.snap_i * N * nmed + m, nmed);
    cells_shared<N, M, COMP, 1>(F, K, z, P);
    P[0] = med ? P[0] : M(0);
    if (med) {
#pragma unroll
      for (int k = 0; k < D; ++k) {
        const Real hi = (Real)z[0][k];
        a.z[k * a.ld + m] = hi;
        if constexpr (COMP) a.z[(D + k) * a.ld + m] = (Real)(z[0][k] - (M)hi);
      }
    }
  }
  const Real hx = tmz_hx(hx0, a.chy, Eup, E), hxd = tmz_hx(hxd0, a.chy, E, Edn);
  const Real hy = tmz_hy(hy0, a.chx, Er, E), hyl = tmz_hy(hyl0, a.chx, E, El);
  const Real curl = (hy - hyl) * a.idx - (hx - hxd) * a.idy;
  Real En = a.ca * E + a.cb * (-(Real)P[0] + curl);
  if (i == 0) En = a.src[a.n + 1] * a.prof[j];
  if (i >= nx) return;
  const int64_t g = j * nx + i;
  a.Hxout[g] = hx;
  if (i == nx - 1) return;  // the Mur column is written by the lane of column nx - 2
  a.Hyout[g] = hy;
  a.Eout[g] = En;
  double *es = a.snap && a.e_out ? a.e_out + a.snap_i * nx * ny + g : nullptr;
  if (es) es[0] = (double)En;
  if (i == nx - 2) {
    const Real Eb = E + a.kmur * (En - Er);
    a.Eout[g + 1] = Eb;
    if (a.probe_out) a.probe_out[(a.n + 1) * ny + j] = (double)Eb;
    if (es) es[1] = (double)Eb;
  }
}

}  // namespace mln
