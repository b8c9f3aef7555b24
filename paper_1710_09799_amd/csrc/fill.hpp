// fill.hpp -- initial states written on the device.
//
// Every solver starts from a state that a few numbers describe (one Bloch
// vector for all medium cells, zero fields, the source sample at cell 0), so
// going back to step 0 is one launch that writes those numbers, not a copy of
// host arrays of the state's size.  A plan holds the buffers of one handle
// (or of all handles of a batch) and their row values in device memory.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <utility>
#include <vector>

#include "devbuf.hpp"

namespace mln {

// element (r, c) of a rows x ld array = c < n ? val[r] : 0 (bytes: 4 or 8 per
// element; val may be NULL when n is 0)
struct FillJob {
  void *p;
  const void *val;
  int64_t rows, ld, n;
  int32_t bytes, pad_;
};

struct FillPlan {
  std::vector<FillJob> jobs;
  // one job; its row values (rows of them, or none for zeros) in FP64,
  // rounded to the job's type
  void add(void *p, int64_t rows, int64_t ld, int64_t n, const std::vector<double> &val, int bytes);
  // one job whose values are in device memory already
  void add_dev(void *p, int64_t rows, int64_t ld, int64_t n, const void *val, int bytes);
  // the jobs of another plan, which is uploaded already and outlives this one
  void add_plan(const FillPlan &o) { jobs.insert(jobs.end(), o.jobs.begin(), o.jobs.end()); }
  // the jobs and their values to the device, in one allocation
  int upload();
  hipError_t run(hipStream_t st) const;

 private:
  std::vector<unsigned char> vals;                 // row values, until upload()
  std::vector<std::pair<size_t, size_t>> pending;  // (job, offset of its values)
  DevBuf dev;
  int64_t most = 0;  // elements of the largest job
};

}  // namespace mln
