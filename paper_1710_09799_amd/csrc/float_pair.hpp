// float_pair.hpp -- rounding an FP64 value to what a pair of floats holds.
#pragma once

#include <cstdint>
#include <cstring>

#include "host_device.hpp"

namespace mln {

// x to the nearest value of 49 bits (ties to even) that is a multiple of the
// smallest float: the float nearest to it and the float of the rest, which
// has a sign, hold it exactly.  The compensated FP32 state is stepped in FP64
// and rounded so after every step, so that a launch boundary, where it is
// stored as a pair, does not change the result.  Adding and taking away 1.5
// 2^(e + 4), e the exponent of x, rounds at 2^(e - 48); its floor 1.5 2^-97
// rounds at 2^-149.
MLN_HD double pair_exact(double x) {
  uint64_t bits;
  std::memcpy(&bits, &x, 8);
  uint32_t hi = ((uint32_t)(bits >> 32) & 0x7ff00000u) + 0x00480000u;
  hi = hi > 0x39e80000u ? hi : 0x39e80000u;
  bits = (uint64_t)hi << 32;
  double m;
  std::memcpy(&m, &bits, 8);
  return (x + m) - m;
}

}  // namespace mln
