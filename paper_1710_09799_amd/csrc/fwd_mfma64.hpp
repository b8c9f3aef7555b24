// fwd_mfma64.hpp -- rotation-route tile kernel of N = 4, 6 in FP64 arithmetic
// with the shared factor on the FP64 matrix cores (plain FP64 and the
// compensated FP32 state, with plain or compensated fields).
//
// A thread that carries a whole cell reads (K - I), 225 or 1225 values, from
// the scalar cache in every step and holds 15 or 35 state values beside it:
// one wavefront per SIMD, which waits for scalar loads most of the time.  Here
// sixteen cells are the columns of one MFMA operand and a cell is four lanes,
// one in each 16-lane row of the wavefront:
//   * v_mfma_f64_16x16x4 reads operand B with row index k = 4 s + g in lane row
//     g, and leaves row 16 t + 4 r + g of the product in accumulator register r
//     of lane row g.  With the state's row 4 s + g in register s of lane row g
//     the product therefore comes back in the layout that the next step reads:
//     no lane ever moves a state value;
//   * the state rows are ordered so that both rows of a rotation pair are
//     registers of one lane (Slots64), and K - I is permuted alike when the
//     launch loads it, once, into registers;
//   * the last 4 rows of N = 6 (36 = 2 x 16 + 4) take v_mfma_f64_4x4x4 (four
//     blocks, the same four rows of K - I against four columns each), so no
//     product is spent on padding beyond the 36th row;
//   * E and H of a cell are carried by its four lanes alike; neighbours' E go
//     through LDS, one barrier per step; P is summed over the four lanes with
//     row swaps, and E is updated and passed on before the product runs.
// The FP64 matrix and vector units share their throughput (measured: a
// v_mfma_f64_16x16x4 takes 64.6 clocks of a SIMD, and every v_fma_f64 beside it
// adds its 4.1), so the step is bound by arithmetic: N = 6, 1311 clocks of
// products and about 450 of rotations and fields per 16 cells, 3.0 us for the
// 256 cells of a compute unit; measured 3.9.  us per step of whole runs with
// the automatic shapes, one cell per thread / this kernel: six levels, 50000
// cells, FP64 11.4 / 4.2, compensated FP32 15.2 / 4.5; 2000 cells, FP64 9.3 /
// 2.4; four levels, FP64, 2000 cells 10.2 / 1.2, 50000 10.3 / 1.8.
#pragma once

#include "fwd_lane.hpp"
#include "medium_cells.hpp"

namespace mln {

typedef double doublex4_t __attribute__((ext_vector_type(4)));

// Order of the state rows: slot s of lane row g holds row[4 s + g] of the
// state (-1: padding).  Pair g + 4 i takes slots 2 i, 2 i + 1; the rows without
// a rotation (2 Q ..) fill the slots without a pair in order.
template <int N>
struct Slots64 {
  static constexpr int D = N * N - 1, Q = N * (N - 1) / 2;
  static constexpr int NP = (Q + 3) / 4;      // rotation pairs per lane
  static constexpr int S = (D + 3) / 4;       // slots per lane
  static constexpr int T = S / 4, R = S % 4;  // 16-row blocks of the product, 4-row blocks behind them
  static_assert(2 * NP <= S, "the pairs fit the slots");
  signed char row[4 * S];
  constexpr Slots64() : row() {
    int r = 2 * Q;
    for (int k = 0; k < 4 * S; ++k) {
      const int s = k / 4, p = k % 4 + 4 * (s / 2);
      row[k] = (signed char)(s < 2 * NP && p < Q ? 2 * p + (s & 1) : (r < D ? r++ : -1));
    }
  }
};
template <int N>
__device__ constexpr Slots64<N> kSlots64{};

// Sum over the four lanes of a cell (lanes l, l + 16, l + 32, l + 48), the same
// bits in all of them.
__device__ __forceinline__ double rows_sum(double x) {
  typedef unsigned uintx2_t __attribute__((ext_vector_type(2)));
  uintx2_t v = __builtin_bit_cast(uintx2_t, x);
  auto lo = __builtin_amdgcn_permlane16_swap(v[0], v[0], false, false);
  auto hi = __builtin_amdgcn_permlane16_swap(v[1], v[1], false, false);
  x = __builtin_bit_cast(double, uintx2_t{lo[0], hi[0]}) + __builtin_bit_cast(double, uintx2_t{lo[1], hi[1]});
  v = __builtin_bit_cast(uintx2_t, x);
  lo = __builtin_amdgcn_permlane32_swap(v[0], v[0], false, false);
  hi = __builtin_amdgcn_permlane32_swap(v[1], v[1], false, false);
  return __builtin_bit_cast(double, uintx2_t{lo[0], hi[0]}) + __builtin_bit_cast(double, uintx2_t{lo[1], hi[1]});
}

constexpr int kMaxMfma64Tile = 256;  // cells per tile

// C groups of 16 cells per wavefront: one leaves a tile of 256 cells 128
// registers, which spill, four a single wavefront per SIMD (six-level FP64, 50000
// cells, tiles of 256: 4.2 us per step, 9.4 with one, 4.8 with four).
constexpr int kMfma64Groups = 2;

// blockDim.x = 4 W / C.  CF: E, H and the
// source are float-float pairs, carried in FP64 between the ends of a launch
// and rounded to a pair in every step.
template <int N, typename Real, bool COMP, bool CF>
__global__ void __launch_bounds__(4 * kMaxMfma64Tile / kMfma64Groups) fwd_mfma64_kernel(FwdArgs<Real> a) {
  constexpr int C = kMfma64Groups;
  using SL = Slots64<N>;
  typedef typename CellType<Real, CF>::type Fld;
  constexpr int D = SL::D, Q = SL::Q, NP = SL::NP, S = SL::S, T = SL::T, R = SL::R;
  // E of cell c of the tile at index c + 1; indices 0 and W + 1 stay zero
  __shared__ Fld sE[2][kMaxMfma64Tile + 2];
  __shared__ Fld sSrc[kMaxStepsPerLaunch];
  __shared__ Fld sMur;
  // read again in every step, where the latency is hidden, to leave the
  // registers to the rest: the constant term in slot order per lane row, and
  // the last rows of the factor
  __shared__ __align__(16) double sC[4][S + S % 2];
  __shared__ double sA4[R > 0 ? R : 1][S][16];
  const ColdArgs<Real> cold = (ColdArgs<Real>)__builtin_amdgcn_kernarg_segment_ptr();
  const int t = threadIdx.x, lane = t & 63, col = lane & 15, g = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int W = (int)(blockDim.x >> 2) * C;
  const int64_t base = (int64_t)blockIdx.x * a.owned - a.halo;
  const int64_t w0 = base + 16 * C * w;  // first cell of the wavefront
  const int64_t i0 = w0 + col;           // the lane's cell of group 0

  const bool any_med = meets_medium(w0, 16 * C, a.mb, a.me);
  const bool all_med = w0 >= a.mb && w0 + 16 * C <= a.me;
  const bool inside = w0 >= 1 && w0 + 16 * C <= a.nx - 1;  // interior cells only
  const bool has_right = base <= a.nx - 1 && base + W > a.nx - 1;

  const signed char *row = kSlots64<N>.row;
  Fld E[C], H[C], Hl[C];
  double z[C][S];
  // per-lane roles of the groups' cells, one bit each: medium, interior (Yee
  // update), cell 0, cell nx-2, cell nx-1
  int medium = 0, interior = 0, source = 0, inner = 0, last = 0;
#pragma unroll
  for (int q = 0; q < C; ++q) {
    const int64_t i = i0 + 16 * q;
    medium |= (i >= a.mb && i < a.me) << q;
    interior |= (i >= 1 && i <= a.nx - 2) << q;
    source |= (i == 0) << q;
    inner |= (i == a.nx - 2) << q;
    last |= (i == a.nx - 1) << q;
    // every load unconditional, from the nearest cell where the lane's own is
    // outside, so that all are in flight at once
    const int64_t ie = i < 0 ? 0 : (i < a.nx ? i : a.nx - 1), ih = ie < a.nx - 1 ? ie : a.nx - 2;
    const int64_t il = ie > 0 ? ie - 1 : 0;
    E[q] = a.Ein[ie];
    H[q] = a.Hin[ih];
    Hl[q] = a.Hin[il];
    if constexpr (CF) {
      E[q] += (Fld)a.Ein[a.nx + ie];
      H[q] += (Fld)a.Hin[a.nx + ih];
      Hl[q] += (Fld)a.Hin[a.nx + il];
    }
  }
  int jr[S];
#pragma unroll
  for (int s = 0; s < S; ++s) jr[s] = row[4 * s + g];
  Real zh[C][S], zl[C][COMP ? S : 1];
#pragma unroll
  for (int q = 0; q < C; ++q) {
    const int64_t i = i0 + 16 * q;
    const int64_t im = nearest_medium(i, a.mb, a.me);
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const int j = jr[s] >= 0 ? jr[s] : 0;
      zh[q][s] = any_med ? a.zin[j * a.ld + im] : Real(0);
      if constexpr (COMP) zl[q][s] = any_med ? a.zin[(D + j) * a.ld + im] : Real(0);
    }
  }

  const double *fK, *fc, *fw, *ft, *fz;
  double p0;
  if constexpr (COMP) {  // the FP64 block
    fK = a.fac.blk64;
    fc = fK + D * D;
    fw = fc + D;
    ft = fw + D;
    fz = ft + Q;
    p0 = cld(fz, D);
  } else {
    fK = a.fac.Km;
    fc = a.fac.cz;
    fw = a.fac.wz;
    ft = a.fac.thdt;
    fz = a.fac.zr;
    p0 = a.fac.p0;
  }
  // K - I as operand A: row of the block in lane & 15 (16x16x4) or lane & 3
  // (4x4x4), column 4 s + g of the permuted factor
  double A[T][S], wz[S];
#pragma unroll
  for (int b = 0; b < T; ++b) {
    const int jm = row[16 * b + col];
#pragma unroll
    for (int s = 0; s < S; ++s) A[b][s] = fK[(jm >= 0 ? jm : 0) * D + (jr[s] >= 0 ? jr[s] : 0)];
#pragma unroll
    for (int s = 0; s < S; ++s) A[b][s] = jm >= 0 && jr[s] >= 0 ? A[b][s] : 0.0;
  }
#pragma unroll
  for (int s = 0; s < S; ++s) wz[s] = fw[jr[s] >= 0 ? jr[s] : 0];
#pragma unroll
  for (int s = 0; s < S; ++s) wz[s] = jr[s] >= 0 ? wz[s] : 0.0;
  for (int x = t; x < 16 * R * S; x += blockDim.x) {
    const int jk = row[4 * (x / 16 % S) + x % 16 / 4], jm = row[16 * T + 4 * (x / (16 * S)) + x % 4];
    (&sA4[0][0][0])[x] = jk >= 0 && jm >= 0 ? fK[jm * D + jk] : 0.0;
  }
  if (t < 4 * S) sC[t & 3][t >> 2] = row[t] >= 0 ? fc[row[t]] : 0.0;
  double zr[2 * NP], th[NP], thmax = 0.0;
#pragma unroll
  for (int i = 0; i < NP; ++i) {  // a row without a rotation has th = 0 and no shift
    const int p = g + 4 * i < Q ? g + 4 * i : 0;
    th[i] = ft[p];
    zr[2 * i] = fz[2 * p];
    zr[2 * i + 1] = fz[2 * p + 1];
  }
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    const bool v = g + 4 * i < Q;
    th[i] = v ? th[i] : 0.0;
    zr[2 * i] = v ? zr[2 * i] : 0.0;
    zr[2 * i + 1] = v ? zr[2 * i + 1] : 0.0;
  }
#pragma unroll
  for (int p = 0; p < Q; ++p) thmax = fmax(thmax, fabs(cld(ft, p)));
  for (int i = t; i < a.nsteps; i += blockDim.x) {
    sSrc[i] = a.src[a.step0 + 1 + i];
    if constexpr (CF) sSrc[i] += (Fld)a.src[a.nt + 1 + a.step0 + 1 + i];
  }
  if (t < 4) sE[t & 1][(t >> 1) ? W + 1 : 0] = Fld(0);
#pragma unroll
  for (int q = 0; q < C; ++q) {
    const int64_t i = i0 + 16 * q;
    E[q] = i >= 0 && i < a.nx ? E[q] : Fld(0);
#pragma unroll
    for (int s = 0; s < S; ++s) {
      double v = (double)zh[q][s];
      if constexpr (COMP) v += (double)zl[q][s];
      z[q][s] = ((medium >> q) & 1) && jr[s] >= 0 ? v : 0.0;
    }
  }
  const int ce = 16 * C * w + col + 1;
  if (g == 0) {
#pragma unroll
    for (int q = 0; q < C; ++q) sE[0][ce + 16 * q] = E[q];
  }
  // whether this tile writes the lane's cell of group q
  auto owned = [&](ColdArgs<Real> c, int q) {
    const int cl = ce - 1 + 16 * q;
    return cl >= c->halo && cl < c->halo + c->owned && i0 + 16 * q >= 0 && i0 + 16 * q < c->nx;
  };
  auto pair = [](Fld x) {
    if constexpr (CF) return pair_exact(x);
    return x;
  };
  auto yee = [&](Fld e, Fld p, Fld h, Fld hl) {
    const Fld f = a.cb * (-p + (h - hl) * a.inv_dx);
    if constexpr (CF) return pair_exact(e + (a.cam1 * e + f));
    return a.ca * e + f;
  };
  int s_snap = (a.snap_next >= a.step0 && a.snap_next < a.step0 + a.nsteps) ? (int)(a.snap_next - a.step0) : -1;
  int snaps = 0;  // snapshots taken in this launch

  for (int s = 0; s < a.nsteps; ++s) {
    const bool snap = s == s_snap;
    int g0 = g, ga = (g << 2) | (lane & 3);
    __asm__ volatile("" : "+v"(g0), "+v"(ga));  // keeps the reads of sC and sA4 in the step loop
    lds_barrier();
    const Fld *e = &sE[s & 1][ce];
    Fld P[C], El[C];
#pragma unroll
    for (int q = 0; q < C; ++q) {
      El[q] = e[16 * q - 1];
      // faces outside the grid are updated too, nothing reads them
      Hl[q] = pair(Hl[q] + a.ch * (E[q] - El[q]));
      H[q] = pair(H[q] + a.ch * (e[16 * q + 1] - E[q]));
      P[q] = 0;
    }
    doublex4_t acc[C][T];
    double acc4[C][R > 0 ? R : 1];
    if (any_med) {
      double em = 0.0;
      bool bad = false;
#pragma unroll
      for (int q = 0; q < C; ++q) {
        const double x = fabs((double)E[q]);
        em = x > em ? x : em;
        bad |= x != x;
      }
      if (__builtin_expect(!wave_any(bad || em * thmax > 0.0625), 1)) {
#pragma unroll
        for (int i = 0; i < NP; ++i) {
#pragma unroll
          for (int q = 0; q < C; ++q) {
            double sn, cm;
            sincm1_series(th[i] * (double)E[q], sn, cm);
            rotate_pair(sn, cm, zr[2 * i], zr[2 * i + 1], z[q][2 * i], z[q][2 * i + 1]);
          }
          if (i % 2) __builtin_amdgcn_sched_barrier(0);  // a few angles at a time: registers
        }
      } else {
#pragma unroll 1
        for (int i = 0; i < NP; ++i) {
          double ti = th[0], r0 = zr[0], r1 = zr[1];
#pragma unroll
          for (int k = 1; k < NP; ++k) {
            ti = k == i ? th[k] : ti;
            r0 = k == i ? zr[2 * k] : r0;
            r1 = k == i ? zr[2 * k + 1] : r1;
          }
#pragma unroll
          for (int q = 0; q < C; ++q) {
            double sn, cm;
            sincm1_wide(ti * (double)E[q], sn, cm);
#pragma unroll
            for (int k = 0; k < NP; ++k)
              if (k == i) rotate_pair(sn, cm, r0, r1, z[q][2 * k], z[q][2 * k + 1]);
          }
        }
      }
      if (__builtin_expect(snap, 0)) {
        const ColdArgs<Real> c = cold_again<Real>(cold);
        double *pop = c->pop_out;
        if (pop) {
          const int64_t nmed = c->me - c->mb;
          const double *map = c->fac.pop, *mapc = c->fac.popc;
#pragma unroll 1
          for (int lv = 0; lv < N; ++lv) {
#pragma unroll
            for (int q = 0; q < C; ++q) {
              double pp = 0.0;
#pragma unroll
              for (int k = 0; k < S; ++k) {
                const int j = row[4 * k + g];
                pp += (j >= 0 ? map[lv * D + j] : 0.0) * z[q][k];
              }
              const double tot = rows_sum(pp) + cld(mapc, lv);
              if (((medium >> q) & 1) && owned(c, q) && (lv & 3) == g)
                pop[((c->snap_i0 + snaps) * N + lv) * nmed + (i0 + 16 * q - c->mb)] = tot;
            }
          }
        }
      }
#pragma unroll
      for (int q = 0; q < C; ++q) {
#pragma unroll
        for (int m = 0; m < T; ++m)
          acc[q][m] = doublex4_t{sC[g0][4 * m], sC[g0][4 * m + 1], sC[g0][4 * m + 2], sC[g0][4 * m + 3]};
#pragma unroll
        for (int m = 0; m < R; ++m) acc4[q][m] = sC[g0][4 * T + m];
      }
#pragma unroll
      for (int q = 0; q < C; ++q) {
        double pw = wz[0] * z[q][0], pv = wz[1] * z[q][1];
#pragma unroll
        for (int k = 2; k < S; k += 2) {
          pw += wz[k] * z[q][k];
          if (k + 1 < S) pv += wz[k + 1 < S ? k + 1 : 0] * z[q][k + 1 < S ? k + 1 : 0];
        }
        P[q] = (Fld)(p0 + rows_sum(pw + pv));
      }
      if (!all_med) {
        int med = medium;
        __asm__ volatile("" : "+v"(med));  // keeps the selects inside this branch
#pragma unroll
        for (int q = 0; q < C; ++q) P[q] = (med >> q) & 1 ? P[q] : Fld(0);
      }
    }
    // E^{n+1} goes to the neighbours before the product, which covers the
    // exchange
    if (inside) {
#pragma unroll
      for (int q = 0; q < C; ++q) E[q] = yee(E[q], P[q], H[q], Hl[q]);
    } else {
      Fld Eold[C];
      const Fld src = sSrc[s];
#pragma unroll
      for (int q = 0; q < C; ++q) {
        Eold[q] = E[q];
        const Fld En = yee(E[q], P[q], H[q], Hl[q]);
        E[q] = (interior >> q) & 1 ? En : ((source >> q) & 1 ? src : E[q]);
      }
#pragma unroll
      for (int q = 0; q < C; ++q) P[q] = Eold[q];
    }
    if (has_right) {  // first-order Mur boundary at cell nx-1 (needs E^{n+1} of cell nx-2)
#pragma unroll
      for (int q = 0; q < C; ++q)
        if (((inner >> q) & 1) && g == 0) sMur = E[q];
      lds_barrier();
#pragma unroll
      for (int q = 0; q < C; ++q)
        if ((last >> q) & 1) {  // never inside: P holds E^n
          const ColdArgs<Real> c = cold_again<Real>(cold);
          E[q] = pair(El[q] + c->kmur * (sMur - P[q]));
          if (c->probe_out && owned(c, q) && g == 0) c->probe_out[c->step0 + s + 1] = (double)E[q];
        }
    }
    if (g == 0) {
#pragma unroll
      for (int q = 0; q < C; ++q) sE[(s & 1) ^ 1][ce + 16 * q] = E[q];
    }
    if (__builtin_expect(snap, 0)) {
      const ColdArgs<Real> c = cold_again<Real>(cold);
      if (c->e_out && g == 0) {
#pragma unroll
        for (int q = 0; q < C; ++q)
          if (owned(c, q)) c->e_out[(c->snap_i0 + snaps) * c->nx + i0 + 16 * q] = (double)E[q];
      }
      s_snap += c->snap_every < kMaxStepsPerLaunch ? (int)c->snap_every : kMaxStepsPerLaunch;
      ++snaps;
    }
    if (any_med) {
#pragma unroll
      for (int k = 0; k < S; ++k) {
        double a4[R > 0 ? R : 1];
#pragma unroll
        for (int m = 0; m < R; ++m) a4[m] = sA4[m][k][ga];
#pragma unroll
        for (int q = 0; q < C; ++q) {
#pragma unroll
          for (int m = 0; m < T; ++m) acc[q][m] = __builtin_amdgcn_mfma_f64_16x16x4f64(A[m][k], z[q][k], acc[q][m], 0, 0, 0);
#pragma unroll
          for (int m = 0; m < R; ++m) acc4[q][m] = __builtin_amdgcn_mfma_f64_4x4x4f64(a4[m], z[q][k], acc4[q][m], 0, 0, 0);
        }
      }
#pragma unroll
      for (int q = 0; q < C; ++q) {
#pragma unroll
        for (int k = 0; k < S; ++k) {
          z[q][k] += k < 4 * T ? acc[q][k < 4 * T ? k / 4 : 0][k % 4] : acc4[q][k >= 4 * T ? k - 4 * T : 0];
          if constexpr (COMP) z[q][k] = pair_exact(z[q][k]);
        }
      }
      if (!all_med) {  // cells beside the medium keep no state
        int med = medium;
        __asm__ volatile("" : "+v"(med));
#pragma unroll
        for (int q = 0; q < C; ++q)
#pragma unroll
          for (int k = 0; k < S; ++k) z[q][k] = (med >> q) & 1 ? z[q][k] : 0.0;
      }
    }
  }
  const ColdArgs<Real> c = cold_again<Real>(cold);
  const int64_t ld = c->ld, mb = c->mb;
  Real *zout = c->zout;
#pragma unroll
  for (int q = 0; q < C; ++q) {
    if (!owned(c, q)) continue;
    const int64_t i = i0 + 16 * q;
    if (g == 0) {
      const Real hi = (Real)E[q];
      c->Eout[i] = hi;
      if constexpr (CF) c->Eout[c->nx + i] = (Real)(E[q] - (Fld)hi);
    }
    if (g == 1 && i <= c->nx - 2) {
      const Real hi = (Real)H[q];
      c->Hout[i] = hi;
      if constexpr (CF) c->Hout[c->nx + i] = (Real)(H[q] - (Fld)hi);
    }
    if ((medium >> q) & 1) {
#pragma unroll
      for (int k = 0; k < S; ++k) {
        const int j = row[4 * k + g];
        if (j >= 0) {
          const Real hi = (Real)z[q][k];
          zout[j * ld + (i - mb)] = hi;
          if constexpr (COMP) zout[(D + j) * ld + (i - mb)] = (Real)(z[q][k] - (double)hi);
        }
      }
    }
  }
}

// W: cells per tile, 64, 128, 192 or 256.
template <int N, typename Real, bool COMP, bool CF>
hipError_t launch_mfma64(int W, const FwdArgs<Real> &a, int64_t nblocks, hipStream_t st) {
  if (W < 64 || W > kMaxMfma64Tile || W % 64 || a.owned + 2 * a.halo > W || a.tape) return hipErrorInvalidValue;
  hipLaunchKernelGGL((fwd_mfma64_kernel<N, Real, COMP, CF>), dim3((unsigned)nblocks), dim3(4 * W / kMfma64Groups), 0, st,
                     a);
  return hipGetLastError();
}

}  // namespace mln
