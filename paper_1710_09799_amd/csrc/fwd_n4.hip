// fwd_n4.hip -- instantiations of the forward kernels for N = 4 levels.
#include <type_traits>

#include "fwd_mfma.hpp"
#include "fwd_mfma64.hpp"
#include "fwd_wave.hpp"

namespace mln {

template <typename Real>
hipError_t launch_fwd_n4(int route, bool comp, bool cf, const FwdArgs<Real> &a, int64_t nblocks, int W, hipStream_t st) {
  if (cf && !comp) return hipErrorInvalidValue;
  if (comp) {
    if constexpr (std::is_same<Real, float>::value) {
      if (route != ROUTE_ROT) return hipErrorInvalidValue;
      return cf ? launch_mfma64<4, float, true, true>(W, a, nblocks, st)
                : launch_mfma64<4, float, true, false>(W, a, nblocks, st);
    }
    return hipErrorInvalidValue;
  }
  switch (route) {
    case ROUTE_ROT:
      if constexpr (sizeof(Real) == 8)
        return launch_mfma64<4, double, false, false>(W, a, nblocks, st);
      else
        hipLaunchKernelGGL((fwd_tile_kernel<4, Real, ROUTE_ROT, false>), dim3((unsigned)nblocks), dim3(W), 0, st, a);
      break;
    case ROUTE_DIAG: hipLaunchKernelGGL((fwd_tile_kernel<4, Real, ROUTE_DIAG, false>), dim3((unsigned)nblocks), dim3(W), 0, st, a); break;
    case ROUTE_RODR: hipLaunchKernelGGL((fwd_tile_kernel<4, Real, ROUTE_RODR, false>), dim3((unsigned)nblocks), dim3(W), 0, st, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <typename Real>
hipError_t launch_fwd_wave_n4(bool comp, int C, const FwdArgs<Real> &a, int64_t nblocks, hipStream_t st) {
  if (C != 1 && C != 2 && C != 4) return hipErrorInvalidValue;
  if constexpr (std::is_same<Real, double>::value) {
    return comp ? hipErrorInvalidValue : launch_mfma64<4, double, false, false>(64 * C, a, nblocks, st);
  } else {
    if (comp) return launch_mfma64<4, float, true, false>(64 * C, a, nblocks, st);
    switch (C) {
      case 1: hipLaunchKernelGGL((fwd_wave_kernel<4, float, false, 1>), dim3((unsigned)nblocks), dim3(64), 0, st, a); break;
      case 2: hipLaunchKernelGGL((fwd_wave_kernel<4, float, false, 2>), dim3((unsigned)nblocks), dim3(64), 0, st, a); break;
      case 4: hipLaunchKernelGGL((fwd_wave_kernel<4, float, false, 4>), dim3((unsigned)nblocks), dim3(64), 0, st, a); break;
    }
    return hipGetLastError();
  }
}

hipError_t launch_fwd_mfma_n4(int nprod, const FwdArgs<float> &a, int64_t nblocks, int W, hipStream_t st) {
  constexpr int D = 4 * 4 - 1;
  if (nprod == 6) {
    const size_t lds = mfma_lds_bytes<D, 6>(W);
    hipError_t e = hipFuncSetAttribute((const void *)fwd_mfma_kernel<4, 6>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((fwd_mfma_kernel<4, 6>), dim3((unsigned)nblocks), dim3(W), lds, st, a);
  } else if (nprod == 3) {
    const size_t lds = mfma_lds_bytes<D, 3>(W);
    hipError_t e = hipFuncSetAttribute((const void *)fwd_mfma_kernel<4, 3>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((fwd_mfma_kernel<4, 3>), dim3((unsigned)nblocks), dim3(W), lds, st, a);
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <typename Real>
hipError_t launch_bloch_n4(int route, bool comp, const BlochArgs<Real> &a, hipStream_t st) {
  const unsigned nb = (unsigned)((a.ncell + 255) / 256);
  if (comp) {
    if constexpr (std::is_same<Real, float>::value) {
      if (route != ROUTE_ROT) return hipErrorInvalidValue;
      hipLaunchKernelGGL((bloch_kernel<4, float, ROUTE_ROT, true>), dim3(nb), dim3(256), 0, st, a);
      return hipGetLastError();
    }
    return hipErrorInvalidValue;
  }
  switch (route) {
    case ROUTE_ROT: hipLaunchKernelGGL((bloch_kernel<4, Real, ROUTE_ROT, false>), dim3(nb), dim3(256), 0, st, a); break;
    case ROUTE_DIAG: hipLaunchKernelGGL((bloch_kernel<4, Real, ROUTE_DIAG, false>), dim3(nb), dim3(256), 0, st, a); break;
    case ROUTE_RODR: hipLaunchKernelGGL((bloch_kernel<4, Real, ROUTE_RODR, false>), dim3(nb), dim3(256), 0, st, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template hipError_t launch_fwd_n4<double>(int, bool, bool, const FwdArgs<double> &, int64_t, int, hipStream_t);
template hipError_t launch_fwd_n4<float>(int, bool, bool, const FwdArgs<float> &, int64_t, int, hipStream_t);
template hipError_t launch_fwd_wave_n4<double>(bool, int, const FwdArgs<double> &, int64_t, hipStream_t);
template hipError_t launch_fwd_wave_n4<float>(bool, int, const FwdArgs<float> &, int64_t, hipStream_t);
template hipError_t launch_bloch_n4<double>(int, bool, const BlochArgs<double> &, hipStream_t);
template hipError_t launch_bloch_n4<float>(int, bool, const BlochArgs<float> &, hipStream_t);

}  // namespace mln
