// cells.hpp -- the rotation-route medium step of several cells per lane,
// N = 2, 3 (the step of rot_cell in fwd_impl.hpp, laid out for kernels that
// fill the chip).
//
// One cell per thread spends as many instructions on fetching the shared
// factor (an LDS read per pair of entries and cell), on testing the angle of
// every rotation and on waiting for them as on the step itself.  Here a lane
// steps C cells together: the factors are wave-uniform scalars (SGPR operands,
// read once for all C cells) or, for K - I of N = 3, which exceeds the scalar
// registers, four registers that DPP row broadcasts read; one test of the
// largest |E| decides the sine series of all rotations, and the C independent
// cells fill the latency of each other's chains.
//
// The compensated FP32 state is stored as float pairs (48 bits) and stepped
// in FP64 here: the pair arithmetic takes ten dependent FP32 instructions per
// addition and twice the products, and with the chip full that is slower than
// FP64 itself (three-level, 2^20 cells, pair arithmetic in this kernel: 8.9e10
// against 1.38e11 cell-updates/s in FP64), which also rounds less.  The state
// is rounded to what a pair holds after every step (pair_exact).
#pragma once

#include "float_pair.hpp"
#include "fwd_impl.hpp"
#include "wide_angle.hpp"

namespace mln {

// A uniform pointer that the compiler takes for a new one: the scalar loads
// through it are neither hoisted out of the step loop nor kept for a later
// use, which would need more scalar registers than there are.
template <typename T>
__device__ __forceinline__ const T *reread(const T *p) {
  __asm__ volatile("" : "+s"(p));
  return p;
}

// Arithmetic type of the medium step.
template <typename Real, bool COMP>
struct CellType {
  typedef Real type;
};
template <>
struct CellType<float, true> {
  typedef double type;
};

__device__ __forceinline__ float pair_exact(float x) { return x; }

// The factors of the step in the arithmetic type M.  Those of N = 2 are held
// in scalar registers for the whole launch: left to itself the compiler reads
// them again in every step and waits for the scalar cache (two-level, 50000
// cells: 4.9e10 against 4.5e10 cell-updates/s).  Those of N = 3 would push the
// series' constants out of the scalar registers (150000 cells: 7.7e10 held,
// 8.1e10 read again).
template <int N, typename M>
struct CellFac {
  static constexpr int D = N * N - 1, Q = N * (N - 1) / 2;
  const M *K;
  M c[D], w[D], th[Q], zr[2 * Q], k2[N == 2 ? D * D : 1];  // k2: K of N = 2
  M p0, thmax;  // thmax: |E| thmax bounds every rotation angle of a cell
  static __device__ __forceinline__ M keep(M x) {
    if constexpr (N == 2) __asm__ volatile("" : "+s"(x));
    return x;
  }
  template <typename Real>
  __device__ __forceinline__ void set(const FacDev<Real> &f) {
    const M *pc, *pw, *pt, *pz;
    M q0;
    if constexpr (sizeof(Real) == sizeof(M)) {
      K = f.Km;
      pc = f.cz;
      pw = f.wz;
      pt = f.thdt;
      pz = f.zr;
      q0 = f.p0;
    } else {  // compensated FP32 state: the FP64 block
      K = f.blk64;
      pc = K + D * D;
      pw = pc + D;
      pt = pw + D;
      pz = pt + Q;
      q0 = cld(pz, D);
    }
    M m = 0;
#pragma unroll
    for (int p = 0; p < Q; ++p) {
      th[p] = keep(cld(pt, p));
      m = th[p] > m ? th[p] : (-th[p] > m ? -th[p] : m);
      zr[2 * p] = keep(cld(pz, 2 * p));
      zr[2 * p + 1] = keep(cld(pz, 2 * p + 1));
    }
#pragma unroll
    for (int i = 0; i < D; ++i) {
      c[i] = keep(cld(pc, i));
      w[i] = keep(cld(pw, i));
    }
    if constexpr (N == 2) {
#pragma unroll
      for (int i = 0; i < D * D; ++i) k2[i] = keep(cld(K, i));
    }
    p0 = keep(q0);
    thmax = m;
  }
};

// sin x and cos x - 1 for |x| <= 1/16 (the first series of sincm1)
__device__ __forceinline__ void sincm1_series(double x, double &s, double &cm1) {
  const double x2 = x * x, x4 = x2 * x2;
  const double s0 = fma(x2, -1.0 / 6.0, 1.0);
  const double s1 = fma(x4, 1.0 / 362880.0, fma(x2, -1.0 / 5040.0, 1.0 / 120.0));
  s = x * fma(x4, s1, s0);
  const double c0 = fma(x2, 1.0 / 24.0, -0.5);
  const double c1 = fma(x4, -1.0 / 3628800.0, fma(x2, 1.0 / 40320.0, -1.0 / 720.0));
  cm1 = x2 * fma(x4, c1, c0);
}
__device__ __forceinline__ void sincm1_series(float x, float &s, float &cm1) {
  const float x2 = x * x;
  s = fmaf(x * x2, fmaf(x2, 1.0f / 120.0f, -1.0f / 6.0f), x);
  cm1 = x2 * fmaf(x2, fmaf(x2, -1.0f / 720.0f, 1.0f / 24.0f), -0.5f);
}

// One rotation pair: y'' = Rot(y) + (Rot - I) zr, formed as (cos - 1)(y + zr)
// + sin (y + zr)': the rounding is that of sin * zr, as when the two products
// are apart.
template <typename M>
__device__ __forceinline__ void rotate_pair(M s, M cm1, M ar, M br, M &a, M &b) {
  const M u = a + ar, v = b + br;
  a += cm1 * u + s * v;
  b += cm1 * v - s * u;
}

// sin x and cos x - 1 of any angle (wide_angle.hpp), out of line; results by
// value, in registers.
static __device__ const double kWide[20] = MLN_WIDE_TABLE;
static __device__ const uint32_t kTurn[40] = MLN_TURN_TABLE;
template <typename M2, typename M>
__device__ __forceinline__ M2 sincm1_any(M x) {
  M2 r;
  if (!wave_any(!(fabs(x) <= M(0.5))))
    medium_angle(x, kWide, r.x, r.y);
  else
    wide_angle(x, kWide, kTurn, r.x, r.y);
  return r;
}
static __device__ __noinline__ double2 sincm1_wide_call(double x) { return sincm1_any<double2>(x); }
static __device__ __noinline__ float2 sincm1_wide_call(float x) { return sincm1_any<float2>(x); }
template <typename M>
__device__ __forceinline__ void sincm1_wide(M x, M &s, M &cm1) {
  const auto r = sincm1_wide_call(x);
  s = r.x;
  cm1 = r.y;
}

template <int N, typename M, int C>
__device__ __forceinline__ void rotate_cells(const CellFac<N, M> &f, const M (&E)[C], M (&z)[C][N * N - 1]) {
#pragma unroll
  for (int p = 0; p < CellFac<N, M>::Q; ++p) {
    const M th = f.th[p], ar = f.zr[2 * p], br = f.zr[2 * p + 1];
#pragma unroll
    for (int c = 0; c < C; ++c) {
      M s, cm1;
      sincm1_series(th * E[c], s, cm1);
      rotate_pair(s, cm1, ar, br, z[c][2 * p], z[c][2 * p + 1]);
    }
  }
}

// Whether a rotation angle of the wavefront may be beyond `limit` (or is NaN).
template <int N, typename M, int C>
__device__ __forceinline__ bool cells_beyond(const CellFac<N, M> &f, const M (&E)[C], M limit) {
  M em = 0;
  bool nan = false;
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const M e = E[c] < 0 ? -E[c] : E[c];
    em = e > em ? e : em;
    nan |= e != e;
  }
  return wave_any(nan || em * f.thmax > limit);
}

// How a kernel evaluates angles beyond the short series.  The branch is cold
// in most runs, but its registers, code and calls shape the step loop around it.
//   inlined: wide_angle at each place;  calls: a call at each place;
//   loop: up to 1/2 rad the series at each place, beyond one call in a loop
//   over the pairs and cells.
// Us a run, inlined / calls / loop: beam of 2048 x 512 cells, three levels, FP64
// 33070 / 34500 / 34300; sweep of 64 problems, FP64 13430 / 13400 / 12740;
// spectral ring, 2048 cells 14520 / 11400 / 11890.  The loop takes 20
// registers more than the calls, a wavefront per SIMD where the budget is
// tight; inlined the FP64 evaluation takes FP32 kernels 45.
enum class Wide { inlined, calls, loop };

template <int N, typename M, int C, Wide HOW>
__device__ __forceinline__ void rotate_cells_wide(const CellFac<N, M> &f, const M (&E)[C], M (&z)[C][N * N - 1]) {
  constexpr int Q = CellFac<N, M>::Q;
  const bool medium = HOW == Wide::loop && !cells_beyond<N, M, C>(f, E, M(0.5));
  M s, cm1;
  if (HOW != Wide::loop || medium) {
#pragma unroll
    for (int p = 0; p < Q; ++p) {
#pragma unroll
      for (int c = 0; c < C; ++c) {
        const M x = f.th[p] * E[c];
        if constexpr (HOW == Wide::inlined)
          wide_angle(x, reread(kWide), reread(kTurn), s, cm1);
        else if constexpr (HOW == Wide::calls)
          sincm1_wide(x, s, cm1);
        else
          medium_angle(x, reread(kWide), s, cm1);
        rotate_pair(s, cm1, f.zr[2 * p], f.zr[2 * p + 1], z[c][2 * p], z[c][2 * p + 1]);
        if constexpr (HOW == Wide::loop) __builtin_amdgcn_sched_barrier(0);  // one angle at a time: registers
      }
    }
  } else {
#pragma unroll 1
    for (int i = 0; i < Q * C; ++i) {
      M x = 0;
#pragma unroll
      for (int k = 0; k < Q * C; ++k)
        if (k == i) x = f.th[k / C] * E[k % C];
      sincm1_wide(x, s, cm1);
#pragma unroll
      for (int k = 0; k < Q * C; ++k) {
        const int p = k / C, c = k % C;
        if (k == i) rotate_pair(s, cm1, f.zr[2 * p], f.zr[2 * p + 1], z[c][2 * p], z[c][2 * p + 1]);
      }
    }
  }
}

// exp(U E dt) of C cells.  |E| thmax <= 1/16 in the whole wavefront (every
// practical field): the short series without a branch per angle.
template <int N, typename M, int C, Wide HOW>
__device__ __forceinline__ void cells_rotate(const CellFac<N, M> &f, const M (&E)[C], M (&z)[C][N * N - 1]) {
  if (__builtin_expect(!cells_beyond<N, M, C>(f, E, M(0.0625)), 1))
    rotate_cells<N, M, C>(f, E, z);
  else
    rotate_cells_wide<N, M, C, HOW>(f, E, z);
}

// Populations of one cell's rotated state, FP64.
template <int N, typename M>
__device__ __forceinline__ void cells_record(const double *map, const double *mapc, const M (&z)[N * N - 1],
                                             double *pop, int64_t stride) {
  constexpr int D = N * N - 1;
#pragma unroll
  for (int a = 0; a < N; ++a) {
    double acc = cld(mapc, a);
#pragma unroll
    for (int j = 0; j < D; ++j) acc += cld(map, a * D + j) * (double)z[j];
    pop[a * stride] = acc;
  }
}

// K - I of N = 3 in registers for the whole launch: entry 16 m + l of the
// row-major factor in register m of lane l of each 16-lane row, so that a DPP
// row broadcast inside the FMA reads any entry with no load at all (a
// v_fmac_f64 with it takes 5.2 clocks against 4.3 with a scalar operand; the
// scalar loads of 64 doubles, which exceed the scalar registers, cost more in
// waits).  All lanes of the wavefront must be active where it is used.
template <int N, typename M>
struct CellK {
  M k[N == 3 ? 4 : 1];
  __device__ __forceinline__ void load(const CellFac<N, M> &f) {
    if constexpr (N == 3) {
#pragma unroll
      for (int m = 0; m < 4; ++m) k[m] = f.K[16 * m + (threadIdx.x & 15)];
    }
  }
};

// One broadcast FMA: acc += (entry J of the lane's 16-lane row of k) * z.
#define MLN_FB64(ACC, K, J, Z) "v_fmac_f64_dpp " ACC ", " K ", " Z " row_newbcast:" #J " row_mask:0xf bank_mask:0xf\n\t"
#define MLN_FB32(ACC, K, J, Z) "v_fmac_f32_dpp " ACC ", " K ", " Z " row_newbcast:" #J " row_mask:0xf bank_mask:0xf\n\t"
// rows 0 and 1 of a 2 x 8 block of two cells: accumulators %0 (row 0, cell a),
// %1 (row 0, cell b), %2 (row 1, cell a), %3 (row 1, cell b), factor %4, states
// %5..%12 (cell a) and %13..%20 (cell b).  The wait states at the head cover
// a factor register that was written just before (a DPP operand).
#define MLN_ROWS2(F)                                                                                           \
  "s_nop 1\n\t" F("%0", "%4", 0, "%5") F("%1", "%4", 0, "%13") F("%2", "%4", 8, "%5") F("%3", "%4", 8, "%13")    \
      F("%0", "%4", 1, "%6") F("%1", "%4", 1, "%14") F("%2", "%4", 9, "%6") F("%3", "%4", 9, "%14")             \
      F("%0", "%4", 2, "%7") F("%1", "%4", 2, "%15") F("%2", "%4", 10, "%7") F("%3", "%4", 10, "%15")           \
      F("%0", "%4", 3, "%8") F("%1", "%4", 3, "%16") F("%2", "%4", 11, "%8") F("%3", "%4", 11, "%16")           \
      F("%0", "%4", 4, "%9") F("%1", "%4", 4, "%17") F("%2", "%4", 12, "%9") F("%3", "%4", 12, "%17")           \
      F("%0", "%4", 5, "%10") F("%1", "%4", 5, "%18") F("%2", "%4", 13, "%10") F("%3", "%4", 13, "%18")         \
      F("%0", "%4", 6, "%11") F("%1", "%4", 6, "%19") F("%2", "%4", 14, "%11") F("%3", "%4", 14, "%19")         \
      F("%0", "%4", 7, "%12") F("%1", "%4", 7, "%20") F("%2", "%4", 15, "%12") F("%3", "%4", 15, "%20")
// the same of one cell: accumulators %0 (row 0), %1 (row 1), factor %2, states %3..%10
#define MLN_ROWS1(F)                                                                                           \
  "s_nop 1\n\t" F("%0", "%2", 0, "%3") F("%1", "%2", 8, "%3") F("%0", "%2", 1, "%4") F("%1", "%2", 9, "%4")      \
      F("%0", "%2", 2, "%5") F("%1", "%2", 10, "%5") F("%0", "%2", 3, "%6") F("%1", "%2", 11, "%6")             \
      F("%0", "%2", 4, "%7") F("%1", "%2", 12, "%7") F("%0", "%2", 5, "%8") F("%1", "%2", 13, "%8")             \
      F("%0", "%2", 6, "%9") F("%1", "%2", 14, "%9") F("%0", "%2", 7, "%10") F("%1", "%2", 15, "%10")
#define MLN_ROWS2_ARGS                                                                                         \
  : "+&v"(a0), "+&v"(b0), "+&v"(a1), "+&v"(b1)                                                                 \
  : "v"(k), "v"(za[0]), "v"(za[1]), "v"(za[2]), "v"(za[3]), "v"(za[4]), "v"(za[5]), "v"(za[6]), "v"(za[7]),     \
    "v"(zb[0]), "v"(zb[1]), "v"(zb[2]), "v"(zb[3]), "v"(zb[4]), "v"(zb[5]), "v"(zb[6]), "v"(zb[7])
#define MLN_ROWS1_ARGS                                                                                         \
  : "+&v"(a0), "+&v"(a1)                                                                                       \
  : "v"(k), "v"(za[0]), "v"(za[1]), "v"(za[2]), "v"(za[3]), "v"(za[4]), "v"(za[5]), "v"(za[6]), "v"(za[7])

__device__ __forceinline__ void rows2(double k, const double (&za)[8], const double (&zb)[8], double &a0, double &a1,
                                      double &b0, double &b1) {
  __asm__(MLN_ROWS2(MLN_FB64) MLN_ROWS2_ARGS);
}
__device__ __forceinline__ void rows2(float k, const float (&za)[8], const float (&zb)[8], float &a0, float &a1,
                                      float &b0, float &b1) {
  __asm__(MLN_ROWS2(MLN_FB32) MLN_ROWS2_ARGS);
}
__device__ __forceinline__ void rows1(double k, const double (&za)[8], double &a0, double &a1) {
  __asm__(MLN_ROWS1(MLN_FB64) MLN_ROWS1_ARGS);
}
__device__ __forceinline__ void rows1(float k, const float (&za)[8], float &a0, float &a1) {
  __asm__(MLN_ROWS1(MLN_FB32) MLN_ROWS1_ARGS);
}
#undef MLN_FB64
#undef MLN_FB32
#undef MLN_ROWS2
#undef MLN_ROWS1
#undef MLN_ROWS2_ARGS
#undef MLN_ROWS1_ARGS

// dP/dt = w.y'' + p0 and y_next = y'' + (K - I) y'' + r of C cells, in groups
// of two (their increments are live beside the states).  PAIR: the state is
// stored as float pairs.
template <int N, typename M, bool PAIR, int C>
__device__ __forceinline__ void cells_shared(const CellFac<N, M> &f, const CellK<N, M> &K, M (&z)[C][N * N - 1],
                                             M (&P)[C]) {
  constexpr int D = N * N - 1;
#pragma unroll
  for (int c = 0; c < C; ++c) P[c] = f.p0;
#pragma unroll
  for (int j = 0; j < D; ++j) {
    const M wj = f.w[j];
#pragma unroll
    for (int c = 0; c < C; ++c) P[c] += wj * z[c][j];
  }
#pragma unroll
  for (int g = 0; g < C; g += 2) {
    const bool two = g + 1 < C;
    const int h = two ? g + 1 : g;
    M da[D], db[D];
    if constexpr (N == 3) {
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        da[2 * m] = db[2 * m] = f.c[2 * m];
        da[2 * m + 1] = db[2 * m + 1] = f.c[2 * m + 1];
        if (two)
          rows2(K.k[m], z[g], z[h], da[2 * m], da[2 * m + 1], db[2 * m], db[2 * m + 1]);
        else
          rows1(K.k[m], z[g], da[2 * m], da[2 * m + 1]);
      }
    } else {
#pragma unroll
      for (int i = 0; i < D; ++i) {
        da[i] = db[i] = f.c[i];
#pragma unroll
        for (int j = 0; j < D; ++j) {
          const M k = f.k2[i * D + j];
          da[i] += k * z[g][j];
          if (two) db[i] += k * z[h][j];
        }
      }
    }
#pragma unroll
    for (int i = 0; i < D; ++i) {
      z[g][i] = PAIR ? pair_exact(z[g][i] + da[i]) : z[g][i] + da[i];
      if (two) z[h][i] = PAIR ? pair_exact(z[h][i] + db[i]) : z[h][i] + db[i];
    }
  }
}

}  // namespace mln
