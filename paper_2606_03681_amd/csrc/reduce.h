// Fixed-order sums of split partials, many outputs in one launch.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tfm {

// out[i] = (accumulate ? out[i] : 0) + sum over z < Z of part[z * stride + i] for i < count.
// With fg set, output i = n fK + k receives sum fg[k] + sb[n] fb[k] instead of the sum, where
// sb[n] = sum over z < Z of bpart[z * bstride + n] (the weight gradient of a product whose input
// was gamma o x-hat + beta, formed from x-hat).  count and the strides are multiples of 4 and
// the pointers 16-byte aligned.
struct ReduceJob {
  const float* part;
  float* out;
  const float* fg;
  const float* fb;
  const float* bpart;
  int64_t count, stride, bstride;
  int32_t Z, fK;
  int32_t og;    // output groups of four per workgroup (set by the launch)
  uint32_t blk0; // first workgroup of the job (set by the launch)
};
constexpr int REDUCE_JOBS = 24;

// The jobs of one backward pass, run as one launch.  add() beyond REDUCE_JOBS is an error the
// launch reports.
struct ReduceList {
  int n = 0;
  bool over = false;
  ReduceJob j[REDUCE_JOBS];
  void add(const float* part, int64_t stride, int Z, int64_t count, float* out) {
    if (n == REDUCE_JOBS) { over = true; return; }
    j[n++] = ReduceJob{part, out, nullptr, nullptr, nullptr, count, stride, 0, Z, 1, 0, 0};
  }
  void add_fold(const float* part, int64_t stride, int Z, int N, int K, float* out,
                const float* bpart, int64_t bstride, const float* fg, const float* fb) {
    if (n == REDUCE_JOBS) { over = true; return; }
    j[n++] = ReduceJob{part, out, fg, fb, bpart, (int64_t)N * K, stride, bstride, Z, K, 0, 0};
  }
};
hipError_t launch_reduce_list(ReduceList& l, int accumulate, hipStream_t s);

}  // namespace tfm
