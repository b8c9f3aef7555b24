// medium_cells.hpp -- where a run of cells meets the medium [mb, me), which may
// be empty.  Plain arithmetic, the same on the host and on the device.
#pragma once

#include <cstdint>

#include "host_device.hpp"

namespace mln {

// whether one of the cells [i0, i0 + n) is a medium cell
MLN_HD bool meets_medium(int64_t i0, int64_t n, int64_t mb, int64_t me) {
  return mb < me && i0 < me && i0 + n > mb;
}

// Column of the state arrays of the medium cell nearest to cell i: what a load
// that no lane skips may read.  Without a medium 0 (a row holds at least one
// element).
MLN_HD int64_t nearest_medium(int64_t i, int64_t mb, int64_t me) {
  return i < mb || me <= mb ? 0 : (i < me ? i - mb : me - mb - 1);
}

}  // namespace mln
