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

#include "fwd_impl.hpp"

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

// A value that a pair of floats holds exactly: multiples of the smallest
// float (the added constant's last place is 2^-149; it changes nothing above
// 2^-44), then 48 bits.  The compensated state is rounded so after every step,
// so that a launch boundary, where it is stored, does not change the result.
__device__ __forceinline__ double pair_exact(double x) {
  const double m = 0x1.8p-97;
  const double r = (x + m) - m;
  return __hiloint2double(__double2hiint(r), __double2loint(r) & ~31);
}
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

// sin x and cos x - 1 of any angle: x = n pi/2 + r, |r| <= pi/4, with pi/2 in
// three parts and fused products (x - n p1 is exact: both are multiples of
// p1's last place or of x's, and the difference is below 2), the Taylor series
// of r to the last bit, and the quadrant.  Written out here because the device
// library's argument reduction, inlined or called, takes registers from the
// step loop (the three-level FP64 kernel needed 200 instead of 160, two
// wavefronts per SIMD instead of three); its constants are read from memory in
// the branch that takes it.
static __device__ const double kWide64[20] = {
    0.63661977236758134308, 0x1.921fb54442d18p+0, 0x1.1a62633145c07p-54, -0x1.f1976b7ed8fbcp-110,
    -1.0 / 6.0, 1.0 / 120.0, -1.0 / 5040.0, 1.0 / 362880.0, -1.0 / 39916800.0, 1.0 / 6227020800.0,
    -1.0 / 1307674368000.0, 1.0 / 355687428096000.0,
    1.0 / 24.0, -1.0 / 720.0, 1.0 / 40320.0, -1.0 / 3628800.0, 1.0 / 479001600.0, -1.0 / 87178291200.0,
    1.0 / 20922789888000.0, -1.0 / 6402373705728000.0};
static __device__ const float kWide32[11] = {
    0.636619772f, 0x1.921fb60000000p+0f, -0x1.777a5c0000000p-25f, -0x1.ee59da0000000p-50f,
    -1.0f / 6.0f, 1.0f / 120.0f, -1.0f / 5040.0f, 1.0f / 362880.0f,
    1.0f / 24.0f, -1.0f / 720.0f, 1.0f / 40320.0f};
__device__ __forceinline__ void sincm1_wide(double x, double &s, double &cm1) {
  const double *k = reread(kWide64);
  const double n = rint(x * cld(k, 0));
  const double r = fma(-n, cld(k, 3), fma(-n, cld(k, 2), fma(-n, cld(k, 1), x)));
  const double r2 = r * r;
  double ps = cld(k, 11), pc = cld(k, 19);
#pragma unroll
  for (int i = 10; i >= 4; --i) ps = fma(ps, r2, cld(k, i));
#pragma unroll
  for (int i = 18; i >= 12; --i) pc = fma(pc, r2, cld(k, i));
  const double sr = fma(r * r2, ps, r), cr = r2 * fma(r2, pc, -0.5);  // sin r, cos r - 1
  const double q = n - 4.0 * floor(0.25 * n);                         // n mod 4 (exact)
  const double c1 = cr + 1.0;
  s = q == 0.0 ? sr : (q == 1.0 ? c1 : (q == 2.0 ? -sr : -c1));
  cm1 = q == 0.0 ? cr : (q == 1.0 ? -sr - 1.0 : (q == 2.0 ? -cr - 2.0 : sr - 1.0));
}
__device__ __forceinline__ void sincm1_wide(float x, float &s, float &cm1) {
  const float *k = reread(kWide32);
  const float n = rintf(x * cld(k, 0));
  const float r = fmaf(-n, cld(k, 3), fmaf(-n, cld(k, 2), fmaf(-n, cld(k, 1), x)));
  const float r2 = r * r;
  float ps = cld(k, 7), pc = cld(k, 10);
#pragma unroll
  for (int i = 6; i >= 4; --i) ps = fmaf(ps, r2, cld(k, i));
#pragma unroll
  for (int i = 9; i >= 8; --i) pc = fmaf(pc, r2, cld(k, i));
  const float sr = fmaf(r * r2, ps, r), cr = r2 * fmaf(r2, pc, -0.5f);
  const float q = n - 4.0f * floorf(0.25f * n);
  const float c1 = cr + 1.0f;
  s = q == 0.0f ? sr : (q == 1.0f ? c1 : (q == 2.0f ? -sr : -c1));
  cm1 = q == 0.0f ? cr : (q == 1.0f ? -sr - 1.0f : (q == 2.0f ? -cr - 2.0f : sr - 1.0f));
}

template <int N, typename M, int C, bool SERIES>
__device__ __forceinline__ void rotate_cells(const CellFac<N, M> &f, const M (&E)[C], M (&z)[C][N * N - 1]) {
#pragma unroll
  for (int p = 0; p < CellFac<N, M>::Q; ++p) {
    const M th = f.th[p], ar = f.zr[2 * p], br = f.zr[2 * p + 1];
#pragma unroll
    for (int c = 0; c < C; ++c) {
      M s, cm1;
      if constexpr (SERIES)
        sincm1_series(th * E[c], s, cm1);
      else
        sincm1_wide(th * E[c], s, cm1);
      rotate_pair(s, cm1, ar, br, z[c][2 * p], z[c][2 * p + 1]);
    }
  }
}

// exp(U E dt) of C cells.  |E| thmax <= 1/16 in the whole wavefront (every
// practical field): the short series without a branch per angle.
template <int N, typename M, int C>
__device__ __forceinline__ void cells_rotate(const CellFac<N, M> &f, const M (&E)[C], M (&z)[C][N * N - 1]) {
  M em = 0;
  bool nan = false;
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const M e = E[c] < 0 ? -E[c] : E[c];
    em = e > em ? e : em;
    nan |= e != e;
  }
  if (__builtin_expect(!wave_any(nan || em * f.thmax > M(0.0625)), 1))
    rotate_cells<N, M, C, true>(f, E, z);
  else
    rotate_cells<N, M, C, false>(f, E, z);
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
