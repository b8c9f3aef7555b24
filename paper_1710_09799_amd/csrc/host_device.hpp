// host_device.hpp -- functions that the kernels and the host (its tests among
// them) share.
#pragma once

#if defined(__HIPCC__)
#include <hip/hip_runtime.h>
#define MLN_HD __host__ __device__ __forceinline__
#else
#define MLN_HD inline
#endif
