// devbuf.hpp -- error reporting and device allocations of the host code.
#pragma once

#include <hip/hip_runtime.h>

#include <string>

#include "../../include/mln.h"

namespace mln {

// Record a message for mln_last_error() and return `code`.
int set_err(int code, const std::string &msg);

#define HIP_TRY(expr)                                                                   \
  do {                                                                                  \
    hipError_t e_ = (expr);                                                             \
    if (e_ != hipSuccess)                                                               \
      return set_err(e_ == hipErrorOutOfMemory ? MLN_ENOMEM : MLN_EHIP,                 \
                     std::string(#expr) + ": " + hipGetErrorString(e_));                \
  } while (0)

// A device allocation owned by the handle.
struct DevBuf {
  void *p = nullptr;
  size_t bytes = 0;
  ~DevBuf() {
    if (p) (void)hipFree(p);
  }
  hipError_t alloc(size_t n) {
    release();
    bytes = n;
    return hipMalloc(&p, n ? n : 1);
  }
  void release() {
    if (p) (void)hipFree(p);
    p = nullptr;
    bytes = 0;
  }
};

}  // namespace mln
