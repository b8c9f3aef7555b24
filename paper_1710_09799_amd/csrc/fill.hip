// fill.hip -- the kernel and the plans of fill.hpp.
#include "fill.hpp"

#include <algorithm>
#include <cstring>

namespace mln {

namespace {

constexpr int kFillThreads = 256, kFillPer = 4;  // consecutive elements per thread
constexpr int64_t kFillBlocks = 2048;            // workgroups of the largest job (8 per compute unit)

template <typename Real>
__device__ __forceinline__ void fill_rows(const FillJob &j) {
  const uint64_t total = (uint64_t)j.rows * (uint64_t)j.ld;
  Real *p = (Real *)j.p;
  const Real *val = (const Real *)j.val;
  for (uint64_t i = ((uint64_t)blockIdx.x * kFillThreads + threadIdx.x) * kFillPer; i < total;
       i += (uint64_t)gridDim.x * kFillThreads * kFillPer) {
    int64_t r = (int64_t)(i / (uint64_t)j.ld), c = (int64_t)(i - (uint64_t)r * (uint64_t)j.ld);
#pragma unroll
    for (int k = 0; k < kFillPer; ++k) {
      if (i + k >= total) break;
      p[i + k] = c < j.n ? val[r] : Real(0);
      if (++c == j.ld) {
        c = 0;
        ++r;
      }
    }
  }
}

// Bound by the stores: a reset of the 2048 x 512 three-level beam writes 101
// MB, one of the 64-problem sweep 140 MB.
__global__ void __launch_bounds__(kFillThreads) fill_kernel(const FillJob *__restrict__ jobs) {
  const FillJob j = jobs[blockIdx.y];
  if (j.bytes == 8)
    fill_rows<double>(j);
  else
    fill_rows<float>(j);
}

}  // namespace

void FillPlan::add(void *p, int64_t rows, int64_t ld, int64_t n, const std::vector<double> &val, int bytes) {
  if (!p || rows <= 0 || ld <= 0) return;
  jobs.push_back(FillJob{p, nullptr, rows, ld, 0, bytes, 0});
  if (val.empty() || n <= 0) return;
  jobs.back().n = n;
  pending.emplace_back(jobs.size() - 1, vals.size());
  vals.resize(vals.size() + (size_t)rows * 8);  // 8-byte slots keep every job's values aligned
  unsigned char *o = vals.data() + pending.back().second;
  for (int64_t i = 0; i < rows; ++i) {
    const double v = i < (int64_t)val.size() ? val[i] : 0.0;
    if (bytes == 8)
      ((double *)o)[i] = v;
    else
      ((float *)o)[i] = (float)v;
  }
}

void FillPlan::add_dev(void *p, int64_t rows, int64_t ld, int64_t n, const void *val, int bytes) {
  if (p && rows > 0 && ld > 0) jobs.push_back(FillJob{p, val, rows, ld, n, bytes, 0});
}

int FillPlan::upload() {
  if (jobs.empty()) return MLN_OK;
  most = 0;
  for (const FillJob &j : jobs) most = std::max<int64_t>(most, j.rows * j.ld);
  const size_t nj = jobs.size() * sizeof(FillJob);
  HIP_TRY(dev.alloc(nj + vals.size()));
  for (const auto &q : pending) jobs[q.first].val = (const unsigned char *)dev.p + nj + q.second;
  std::vector<unsigned char> all(nj + vals.size());
  std::memcpy(all.data(), jobs.data(), nj);
  if (!vals.empty()) std::memcpy(all.data() + nj, vals.data(), vals.size());
  HIP_TRY(hipMemcpy(dev.p, all.data(), all.size(), hipMemcpyHostToDevice));
  vals.clear();
  pending.clear();
  return MLN_OK;
}

hipError_t FillPlan::run(hipStream_t st) const {
  const int64_t per = (int64_t)kFillThreads * kFillPer;
  const unsigned nb = (unsigned)std::min<int64_t>(kFillBlocks, std::max<int64_t>(1, (most + per - 1) / per));
  for (size_t k = 0; k < jobs.size(); k += 65535) {  // the launch grid's limit in y
    const unsigned nj = (unsigned)std::min<size_t>(65535, jobs.size() - k);
    hipLaunchKernelGGL(fill_kernel, dim3(nb, nj), dim3(kFillThreads), 0, st, (const FillJob *)dev.p + k);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace mln
