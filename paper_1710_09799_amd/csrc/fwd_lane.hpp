// fwd_lane.hpp -- rotation-route tile kernel for grids that fill the chip:
// one wavefront per tile, C consecutive cells per lane (tile W = 64 C), N = 2,
// 3, in the plain and the compensated state.
//
// The one-cell-per-thread tile kernel passes two workgroup barriers and two
// LDS exchanges per step and reads the shared factor from LDS for every cell.
// Here a lane's neighbours are its own registers except at its two ends,
// which a wavefront shift (DPP) passes on; the H face left of the lane's first
// cell is a private copy, updated with the operands its owner uses, so a step
// has no barrier and no exchange through LDS (which holds the launch's source
// samples in the tiles at the grid's ends); and the medium step takes the C
// cells together (cells.hpp).  Tiles inside the grid whose cells are all medium
// (or all vacuum) take no per-cell test.  Temporal blocking as in the other
// tile kernels: nsteps <= halo steps per launch, the owned central cells
// written back.
//
// The scalar registers bound the step loop (they hold the factors, the series'
// constants and the update coefficients), so what only a recording step, the
// tape or an edge tile needs is read from the argument block again when it is
// needed (cold), not kept.
#pragma once

#include "cells.hpp"
#include "fwd_wave.hpp"

namespace mln {

// C consecutive values, in accesses of up to 16 bytes per lane (the rows need
// no alignment beyond the value's own: unaligned global accesses are whole)
template <typename Real>
struct RunVec;
template <>
struct RunVec<double> {
  typedef double type __attribute__((ext_vector_type(2), aligned(8)));
  static constexpr int n = 2;
};
template <>
struct RunVec<float> {
  typedef float type __attribute__((ext_vector_type(4), aligned(4)));
  static constexpr int n = 4;
};
template <int C, typename Real>
__device__ __forceinline__ void load_run(const Real *p, Real (&v)[C]) {
  constexpr int n = RunVec<Real>::n;
#pragma unroll
  for (int j = 0; j + n <= C; j += n) {
    const auto q = *(const typename RunVec<Real>::type *)(p + j);
#pragma unroll
    for (int k = 0; k < n; ++k) v[j + k] = q[k];
  }
#pragma unroll
  for (int j = C / n * n; j < C; ++j) v[j] = p[j];
}
template <int C, typename Real>
__device__ __forceinline__ void store_run(Real *p, const Real (&v)[C]) {
  constexpr int n = RunVec<Real>::n;
#pragma unroll
  for (int j = 0; j + n <= C; j += n) {
    typename RunVec<Real>::type q;
#pragma unroll
    for (int k = 0; k < n; ++k) q[k] = v[j + k];
    *(typename RunVec<Real>::type *)(p + j) = q;
  }
#pragma unroll
  for (int j = C / n * n; j < C; ++j) p[j] = v[j];
}

// The argument block in constant memory, for reads outside the hot path.
template <typename Real>
using ColdArgs = const __attribute__((address_space(4))) FwdArgs<Real> *;
template <typename Real>
__device__ __forceinline__ ColdArgs<Real> cold_again(ColdArgs<Real> p) {
  __asm__ volatile("" : "+s"(p));
  return p;
}

// step0, nsteps: the launch's steps; s_snap, si0: its first recording step
// (an index within the launch, -1: none) and that snapshot's number.
template <int N, typename Real, bool COMP, int C>
__device__ __forceinline__ void lane_tile(const FwdArgs<Real> &a, ColdArgs<Real> cold, int64_t tile, int64_t step0,
                                          int nsteps, int s_snap, int64_t si0) {
  typedef typename CellType<Real, COMP>::type M;
  constexpr int D = N * N - 1;
  constexpr int W = 64 * C;
  const int lane = threadIdx.x & 63;
  const int64_t base = tile * a.owned - a.halo;
  const int64_t g0 = base + (int64_t)lane * C;
  __shared__ Real sSrc[kMaxStepsPerLaunch];
  CellFac<N, M> F;
  F.set(a.fac);
  CellK<N, M> K;
  K.load(F);
  const bool inside = base >= 1 && base + W <= a.nx - 1;  // no source, no boundary, no cell beyond the grid
  const bool any_med = base < a.me && base + W > a.mb;
  const bool all_med = base >= a.mb && base + W <= a.me;

  Real E[C], H[C];
  M z[C][D];
  Real Hl = 0;
  // the compensated state's floats, all under way before the first is summed
  Real zh[COMP ? D : 1][C], zl[COMP ? D : 1][C];
  if (inside && (all_med || !any_med)) {  // whole runs of C cells
    load_run<C>(a.Ein + g0, E);
    load_run<C>(a.Hin + g0, H);
    Hl = a.Hin[g0 - 1];
    if constexpr (COMP) {
      if (all_med) {
#pragma unroll
        for (int i = 0; i < D; ++i) {
          load_run<C>(a.zin + i * a.ld + (g0 - a.mb), zh[i]);
          load_run<C>(a.zin + (D + i) * a.ld + (g0 - a.mb), zl[i]);
        }
      } else {
#pragma unroll
        for (int i = 0; i < D; ++i)
#pragma unroll
          for (int j = 0; j < C; ++j) zh[i][j] = zl[i][j] = 0;
      }
    } else {
#pragma unroll
      for (int i = 0; i < D; ++i) {
        Real t[C];
#pragma unroll
        for (int j = 0; j < C; ++j) t[j] = 0;
        if (all_med) load_run<C>(a.zin + i * a.ld + (g0 - a.mb), t);
#pragma unroll
        for (int j = 0; j < C; ++j) z[j][i] = t[j];
      }
    }
  } else {
    if (g0 - 1 >= 0 && g0 - 1 <= a.nx - 2) Hl = a.Hin[g0 - 1];
#pragma unroll
    for (int j = 0; j < C; ++j) {
      const int64_t g = g0 + j;
      const bool med = g >= a.mb && g < a.me;
      E[j] = (g >= 0 && g < a.nx) ? a.Ein[g] : Real(0);
      H[j] = (g >= 0 && g <= a.nx - 2) ? a.Hin[g] : Real(0);
#pragma unroll
      for (int i = 0; i < D; ++i) {
        if constexpr (COMP) {
          zh[i][j] = med ? a.zin[i * a.ld + (g - a.mb)] : Real(0);
          zl[i][j] = med ? a.zin[(D + i) * a.ld + (g - a.mb)] : Real(0);
        } else {
          z[j][i] = med ? a.zin[i * a.ld + (g - a.mb)] : Real(0);
        }
      }
    }
    for (int i = lane; i < nsteps; i += 64) sSrc[i] = a.src[step0 + 1 + i];
    // (one wavefront: orders the writes before the other lanes' reads)
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
  if constexpr (COMP) {
#pragma unroll
    for (int j = 0; j < C; ++j)
#pragma unroll
      for (int i = 0; i < D; ++i) z[j][i] = (M)zh[i][j] + (M)zl[i][j];
  }
  // per-lane roles of the C cells, one bit each: medium, interior (Yee
  // update), cell 0, cell nx-1
  int medium = 0, interior = 0, source = 0, last = 0;
#pragma unroll
  for (int j = 0; j < C; ++j) {
    const int64_t g = g0 + j;
    medium |= (g >= a.mb && g < a.me) << j;
    interior |= (g >= 1 && g <= a.nx - 2) << j;
    source |= (g == 0) << j;
    last |= (g == a.nx - 1) << j;
  }
  const int t0 = lane * C;
  const int s_tape = !a.tape ? nsteps : (int)(a.tape_step0 <= step0 ? 0 : a.tape_step0 - step0 < nsteps ? a.tape_step0 - step0 : nsteps);
  int snaps = 0;  // snapshots taken in this launch

  for (int s = 0; s < nsteps; ++s) {
    const bool snap = s == s_snap;
    const Real El = wave_shift<kDppWaveShr1>(E[C - 1]);
    const Real Er = wave_shift<kDppWaveShl1>(E[0]);
    // H^{n+1/2}; faces outside the grid are updated too, nothing reads them
    Hl += a.ch * (E[0] - El);
#pragma unroll
    for (int j = 0; j < C; ++j) H[j] += a.ch * ((j + 1 < C ? E[j + 1] : Er) - E[j]);
    M P[C];
#pragma unroll
    for (int j = 0; j < C; ++j) P[j] = 0;
    if (any_med) {
      if (s >= s_tape) {
        const ColdArgs<Real> c = cold_again<Real>(cold);
        const int64_t row = step0 + s - c->tape_step0;
#pragma unroll
        for (int j = 0; j < C; ++j)
          if (((medium >> j) & 1) && t0 + j >= c->halo && t0 + j < c->halo + c->owned) {
            Real *tp = c->tape + row * (D + 1) * c->ld + (g0 + j - c->mb);
#pragma unroll
            for (int i = 0; i < D; ++i) tp[i * c->ld] = (Real)z[j][i];
            tp[D * c->ld] = E[j];
          }
      }
      M Em[C];
#pragma unroll
      for (int j = 0; j < C; ++j) Em[j] = (M)E[j];
      cells_rotate<N, M, C, C == 4 && sizeof(M) == 8 ? Wide::loop : Wide::calls>(F, Em, z);
      if (__builtin_expect(snap, 0)) {
        const ColdArgs<Real> c = cold_again<Real>(cold);
        const int64_t nmed = c->me - c->mb;
        double *pop = c->pop_out;
        if (pop) {
#pragma unroll
          for (int j = 0; j < C; ++j)
            if (((medium >> j) & 1) && t0 + j >= c->halo && t0 + j < c->halo + c->owned)
              cells_record<N, M>(c->fac.pop, c->fac.popc, z[j], pop + (si0 + snaps) * N * nmed + (g0 + j - c->mb),
                                 nmed);
        }
      }
      cells_shared<N, M, COMP, C>(F, K, z, P);
      if (!all_med) {  // cells beside the medium keep no state and no polarisation
#pragma unroll
        for (int j = 0; j < C; ++j) {
          int med = (medium >> j) & 1;
          __asm__ volatile("" : "+v"(med));  // keeps the selects inside this branch
          P[j] = med ? P[j] : M(0);
#pragma unroll
          for (int i = 0; i < D; ++i) z[j][i] = med ? z[j][i] : M(0);
        }
      }
    }
    if (inside) {
#pragma unroll
      for (int j = 0; j < C; ++j)
        E[j] = a.ca * E[j] + a.cb * (-(Real)P[j] + (H[j] - (j ? H[j ? j - 1 : 0] : Hl)) * a.inv_dx);
    } else {
      Real Eold[C];
      const Real src = sSrc[s];
#pragma unroll
      for (int j = 0; j < C; ++j) {
        Eold[j] = E[j];
        const Real En = a.ca * E[j] + a.cb * (-(Real)P[j] + (H[j] - (j ? H[j ? j - 1 : 0] : Hl)) * a.inv_dx);
        E[j] = (interior >> j) & 1 ? En : ((source >> j) & 1 ? src : E[j]);
      }
      // first-order Mur boundary at cell nx-1 (needs E^n and E^{n+1} of nx-2)
      const Real Eln = wave_shift<kDppWaveShr1>(E[C - 1]);
#pragma unroll
      for (int j = 0; j < C; ++j)
        if ((last >> j) & 1) {
          const ColdArgs<Real> c = cold_again<Real>(cold);
          const Real prev_old = j ? Eold[j ? j - 1 : 0] : El, prev_new = j ? E[j ? j - 1 : 0] : Eln;
          E[j] = prev_old + c->kmur * (prev_new - Eold[j]);
          if (c->probe_out && t0 + j >= c->halo && t0 + j < c->halo + c->owned)
            c->probe_out[step0 + s + 1] = (double)E[j];
        }
    }
    if (__builtin_expect(snap, 0)) {
      const ColdArgs<Real> c = cold_again<Real>(cold);
      if (c->e_out) {
#pragma unroll
        for (int j = 0; j < C; ++j)
          if (g0 + j >= 0 && g0 + j < c->nx && t0 + j >= c->halo && t0 + j < c->halo + c->owned)
            c->e_out[(si0 + snaps) * c->nx + g0 + j] = (double)E[j];
      }
      s_snap += c->snap_every < kMaxStepsPerLaunch ? (int)c->snap_every : kMaxStepsPerLaunch;
      ++snaps;
    }
  }

  const ColdArgs<Real> c = cold_again<Real>(cold);
  const int64_t ld = c->ld, mb = c->mb;
  const int halo = c->halo, owned = c->owned;
  Real *zout = c->zout;
  if (inside && (all_med || !any_med) && halo % C == 0 && owned % C == 0) {
    // the lane's cells are owned all or none
    if (t0 >= halo && t0 < halo + owned) {
      store_run<C>(c->Eout + g0, E);
      store_run<C>(c->Hout + g0, H);
      if (all_med) {
#pragma unroll
        for (int i = 0; i < D; ++i) {
          Real t[C], tl[C];
#pragma unroll
          for (int j = 0; j < C; ++j) {
            t[j] = (Real)z[j][i];
            tl[j] = COMP ? (Real)(z[j][i] - (M)t[j]) : Real(0);
          }
          store_run<C>(zout + i * ld + (g0 - mb), t);
          if constexpr (COMP) store_run<C>(zout + (D + i) * ld + (g0 - mb), tl);
        }
      }
    }
    return;
  }
#pragma unroll
  for (int j = 0; j < C; ++j) {
    const int64_t g = g0 + j;
    if (g < 0 || g >= c->nx || t0 + j < halo || t0 + j >= halo + owned) continue;
    c->Eout[g] = E[j];
    if (g <= c->nx - 2) c->Hout[g] = H[j];
    if ((medium >> j) & 1) {
#pragma unroll
      for (int i = 0; i < D; ++i) {
        const Real t = (Real)z[j][i];
        zout[i * ld + (g - mb)] = t;
        if constexpr (COMP) zout[(D + i) * ld + (g - mb)] = (Real)(z[j][i] - (M)t);
      }
    }
  }
}

// Register budget in wavefronts per SIMD: with four cells per lane the
// three-level FP64 step takes two (190 registers; compiled for three it
// spills), else four.
template <int N, typename Real, bool COMP, int C>
constexpr int lane_waves() {
  return N == 3 && C >= 3 && (COMP || sizeof(Real) == 8) ? 2 : 4;
}

template <int N, typename Real, bool COMP, int C>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(lane_waves<N, Real, COMP, C>(), 8)))
fwd_lane_kernel(FwdArgs<Real> a) {
  const ColdArgs<Real> cold = (ColdArgs<Real>)__builtin_amdgcn_kernarg_segment_ptr();
  const int s_snap = (a.snap_next >= a.step0 && a.snap_next < a.step0 + a.nsteps) ? (int)(a.snap_next - a.step0) : -1;
  lane_tile<N, Real, COMP, C>(a, cold, blockIdx.x, a.step0, a.nsteps, s_snap, a.snap_i0);
}

// W = 64, 128, 192 or 256 cells per tile
template <int N, typename Real, bool COMP>
hipError_t launch_lane(int W, const FwdArgs<Real> &a, int64_t nblocks, hipStream_t st) {
  const dim3 grid((unsigned)nblocks), block(64);
  switch (W) {
    case 64: hipLaunchKernelGGL((fwd_lane_kernel<N, Real, COMP, 1>), grid, block, 0, st, a); break;
    case 128: hipLaunchKernelGGL((fwd_lane_kernel<N, Real, COMP, 2>), grid, block, 0, st, a); break;
    case 192: hipLaunchKernelGGL((fwd_lane_kernel<N, Real, COMP, 3>), grid, block, 0, st, a); break;
    case 256: hipLaunchKernelGGL((fwd_lane_kernel<N, Real, COMP, 4>), grid, block, 0, st, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace mln
