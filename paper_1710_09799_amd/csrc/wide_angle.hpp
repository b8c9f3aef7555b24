// wide_angle.hpp -- sin x and cos x - 1 of any finite angle, for the branch
// that a wavefront takes when one of its angles lies beyond the short series.
// The same source serves the kernels and, on the host, their tests.
//
// The angle is reduced to n pi/2 + r + rl, |r| <= pi/4 (a little more near
// 2^45), rl the rounding of r, and r is summed by its Taylor series.  Single-precision angles go the same way
// in FP64 and are rounded once, at the end.
//   |x| < 2^45: Cody and Waite (Software Manual for the Elementary Functions,
//     1980): n pi/2 is taken off in three parts of pi/2, here by fused
//     products.
//   beyond: Payne and Hanek (Radian Reduction for Trigonometric Functions,
//     SIGNUM Newsletter 18, 1983): of the angle's 53-bit integer times 1/(2 pi)
//     only the fraction of a turn is formed, from the 192 bits of 1/(2 pi) that
//     it depends on.
// Absolute errors against long double from 1/16 to the largest angle: FP64 sin
// 6.1e-17 (a correctly rounded sine: 5.6e-17), cos - 1 1.7e-16, of values up to 2
// (as -2 sin^2(x/2) from a library sine: 3.3e-16); FP32 3.0e-8 and 6.0e-8 (1.8e-7).
//
// Most kernels call it out of line (sincm1_wide): inlined, its registers cost
// the step loop a wavefront per SIMD (the device library's sine alike: 200
// instead of 160 in the three-level FP64 kernel).
#pragma once

#include <cmath>
#include <cstdint>
#include <cstring>

#include "host_device.hpp"

namespace mln {

// 2/pi; pi/2 in three parts; the sine's coefficients of r^3 .. r^17; those of
// the cosine of r^4 .. r^18
#define MLN_WIDE_TABLE                                                                                        \
  {0.63661977236758134308, 0x1.921fb54442d18p+0, 0x1.1a62633145c07p-54, -0x1.f1976b7ed8fbcp-110, -1.0 / 6.0,   \
   1.0 / 120.0, -1.0 / 5040.0, 1.0 / 362880.0, -1.0 / 39916800.0, 1.0 / 6227020800.0, -1.0 / 1307674368000.0,  \
   1.0 / 355687428096000.0, 1.0 / 24.0, -1.0 / 720.0, 1.0 / 40320.0, -1.0 / 3628800.0, 1.0 / 479001600.0,      \
   -1.0 / 87178291200.0, 1.0 / 20922789888000.0, -1.0 / 6402373705728000.0}
// 1/(2 pi) in binary, 32 bits a word, after 32 zero bits
#define MLN_TURN_TABLE                                                                                        \
  {0x00000000u, 0x28be60dbu, 0x9391054au, 0x7f09d5f4u, 0x7d4d3770u, 0x36d8a566u, 0x4f10e410u, 0x7f9458eau,     \
   0xf7aef158u, 0x6dc91b8eu, 0x909374b8u, 0x01924bbau, 0x82746487u, 0x3f877ac7u, 0x2c4a69cfu, 0xba208d7du,     \
   0x4baed121u, 0x3a671c09u, 0xad17df90u, 0x4e64758eu, 0x60d4ce7du, 0x272117e2u, 0xef7e4a0eu, 0xc7fe25ffu,     \
   0xf7816603u, 0xfbcbc462u, 0xd6829b47u, 0xdb4d9fb3u, 0xc9f2c26du, 0xd3d18fd9u, 0xa797fa8bu, 0x5d49eeb1u,     \
   0xfaf97c5eu, 0xcf41ce7du, 0xe294a4bau, 0x9afed7ecu, 0x47e35742u, 0x1580cc11u, 0xbf1edaeau, 0xfc33ef08u}

// sin x and cos x - 1, |x| <= 1/2: the series alone, in x's own precision.
MLN_HD void medium_angle(double x, const double *k, double &s, double &cm1) {
  const double x2 = x * x;
  double ps = k[11], pc = k[19];
#pragma unroll
  for (int i = 10; i >= 4; --i) ps = fma(ps, x2, k[i]);
#pragma unroll
  for (int i = 18; i >= 12; --i) pc = fma(pc, x2, k[i]);
  s = fma(x * x2, ps, x);
  cm1 = x2 * fma(x2, pc, -0.5);
}
MLN_HD void medium_angle(float x, const double *, float &s, float &cm1) {
  const float x2 = x * x;
  const float ps = fmaf(fmaf(fmaf(1.0f / 362880.0f, x2, -1.0f / 5040.0f), x2, 1.0f / 120.0f), x2, -1.0f / 6.0f);
  const float pc = fmaf(fmaf(fmaf(-1.0f / 3628800.0f, x2, 1.0f / 40320.0f), x2, -1.0f / 720.0f), x2, 1.0f / 24.0f);
  s = fmaf(x * x2, ps, x);
  cm1 = x2 * fmaf(x2, pc, -0.5f);
}

// x = n pi/2 + r + rl (r NaN for NaN and infinities)
MLN_HD void reduce_angle(double x, const double *k, const uint32_t *turn, double &n, double &r, double &rl) {
  if (fabs(x) < 0x1p45) {
    n = rint(x * k[0]);
    const double t = fma(-n, k[1], x);  // exact
    r = fma(-n, k[2], t);
    rl = fma(-n, k[3], fma(-n, k[2], t - r));
    return;
  }
  typedef unsigned __int128 u128;
  uint64_t bits;
  std::memcpy(&bits, &x, 8);
  const int e = (int)(bits >> 52 & 0x7ff);
  if (e == 0x7ff) {
    n = rl = 0.0;
    r = x - x;
    return;
  }
  // |x| = m 2^j; the first j bits of the fraction 1/(2 pi) give whole turns
  const uint64_t m = (bits & 0xfffffffffffffull) | 0x10000000000000ull;
  const int p = e - 1075 + 32, word = p >> 5, sh = p & 31;
  u128 f = 0, carry = 0;  // upper 128 bits of m times the 192 bits from p on, modulo a turn
#pragma unroll 1
  for (int i = 5; i >= 0; --i) {
    const uint32_t w = (uint32_t)((((uint64_t)turn[word + i] << 32) | turn[word + i + 1]) << sh >> 32);
    carry += (u128)w * m;
    f = f >> 32 | carry << 96;
    carry >>= 32;
  }
  // the nearest quadrant, and the rest, g 2^-62 of one, in two parts
  const uint64_t hi = (uint64_t)(f >> 64), q = (hi + (1ull << 61)) >> 62;
  const int64_t g = (int64_t)(hi - (q << 62));
  const double sign = bits >> 63 ? -0x1p-62 : 0x1p-62;
  const double gh = (double)g, gl = (double)(g - (int64_t)gh) + (double)(uint64_t)f * 0x1p-64;
  const double a = sign * gh;
  n = bits >> 63 ? -(double)q : (double)q;
  r = a * k[1];
  rl = fma(a, k[2], fma(a, k[1], -r)) + sign * gl * k[1];
}

// sin x and cos x - 1; k: MLN_WIDE_TABLE, turn: MLN_TURN_TABLE.
MLN_HD void wide_angle(double x, const double *k, const uint32_t *turn, double &s, double &cm1) {
  double n, r, rl;
  reduce_angle(x, k, turn, n, r, rl);
  const double r2 = r * r, r3 = r * r2;
  double ps = k[11], pc = k[19];
#pragma unroll
  for (int i = 10; i >= 5; --i) ps = fma(ps, r2, k[i]);
#pragma unroll
  for (int i = 18; i >= 12; --i) pc = fma(pc, r2, k[i]);
  // cos r - 1 = -r^2/2 + t, sin r = r - r^3/6 + r^5 ps; what the leading sums
  // and the powers of r round off goes to the small terms, and so does rl
  const double r2l = fma(r, r, -r2), r3l = fma(r, r2, -r3) + r * r2l;
  const double v = fma(r3, k[4], r);
  const double t = fma(r2 * r2, pc, -fma(0.5, r2l, v * rl));
  const double cr = fma(-0.5, r2, t);
  const double w = fma(-0.5, r2, 1.0), c1 = w + (fma(-0.5, r2, 1.0 - w) + t);
  const double sr = v + (fma(r3, k[4], r - v) + fma(r3 * r2, ps, fma(r3l, k[4], fma(cr, rl, rl))));
  const double q = n - 4.0 * floor(0.25 * n);  // n mod 4 (exact)
  s = q == 0.0 ? sr : (q == 1.0 ? c1 : (q == 2.0 ? -sr : -c1));
  cm1 = q == 0.0 ? cr : (q == 1.0 ? -sr - 1.0 : (q == 2.0 ? -cr - 2.0 : sr - 1.0));
}
MLN_HD void wide_angle(float x, const double *k, const uint32_t *turn, float &s, float &cm1) {
  double ds, dc;
  wide_angle((double)x, k, turn, ds, dc);
  s = (float)ds;
  cm1 = (float)dc;
}

}  // namespace mln
