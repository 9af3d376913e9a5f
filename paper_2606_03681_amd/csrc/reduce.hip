// Sums of split partials (declarations in reduce.h).
//
// A backward pass ends with one sum per parameter block: six weight matrices, six biases and
// the norm parameters.  As a launch each they cost 28 launches (5 to 8 us apiece, more than the
// data they move on tables of a few thousand cells); as jobs of one grid they cost one.  Each
// workgroup owns 4 og consecutive outputs of one job; its 256 / og groups of threads take
// interleaved partials, four loads in flight each, and their sums are added in a fixed tree
// (bitwise reproducible).  og is 32 where a job has enough outputs to fill the chip (wide rows,
// coalesced 512-byte reads) and 8 or 2 where it has few outputs and many partials (the norm
// parameters: thousands of partial rows of 2E floats), so that no thread walks a long chain.
#include "reduce.h"

namespace tfm {

namespace {

struct ReduceArgs {
  ReduceJob j[REDUCE_JOBS];
  int32_t n, accumulate;
};

__device__ __forceinline__ float4 add4(const float4& a, const float4& b) {
  return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w);
}

__global__ __launch_bounds__(256) void k_reduce_list(ReduceArgs a) {
  __shared__ float4 red[256];
  __shared__ float sbr[256];
  int ji = 0;
  while (ji + 1 < a.n && blockIdx.x >= a.j[ji + 1].blk0) ++ji;
  const ReduceJob& J = a.j[ji];
  const int tid = threadIdx.x, og = J.og, nz = 256 / og;
  const int o = tid % og, zg = tid / og;
  const int64_t i0 = (int64_t)(blockIdx.x - J.blk0) * og * 4;
  const int64_t i4 = i0 + 4 * o;
  const bool on = i4 < J.count;
  float4 s[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) s[u] = make_float4(0.f, 0.f, 0.f, 0.f);
  if (on) {
    const float* p = J.part + i4;
    int z = zg;
    for (; z + 3 * nz < J.Z; z += 4 * nz) {
      float4 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        v[u] = *reinterpret_cast<const float4*>(p + (int64_t)(z + u * nz) * J.stride);
#pragma unroll
      for (int u = 0; u < 4; ++u) s[u] = add4(s[u], v[u]);
    }
    for (int u = 0; z < J.Z; z += nz, ++u) {
      const float4 v = *reinterpret_cast<const float4*>(p + (int64_t)z * J.stride);
      if (u == 0) s[0] = add4(s[0], v);
      else if (u == 1) s[1] = add4(s[1], v);
      else s[2] = add4(s[2], v);
    }
  }
  red[tid] = add4(add4(s[0], s[1]), add4(s[2], s[3]));
  __syncthreads();
  for (int h = nz >> 1; h > 0; h >>= 1) {
    if (zg < h) red[tid] = add4(red[tid], red[tid + h * og]);
    __syncthreads();
  }
  const float4 t = red[tid % og];
  float tv[4] = {t.x, t.y, t.z, t.w};
  if (J.fg) {
    // bias sums of the rows this workgroup's outputs lie in (at most two for K >= 4 og)
    const int64_t last = (i0 + 4 * og < J.count ? i0 + 4 * og : J.count) - 1;
    const int n0 = (int)(i0 / J.fK), n1 = (int)(last / J.fK);
    for (int n = n0; n <= n1; ++n) {
      float b = 0.f;
      for (int z = tid; z < J.Z; z += 256) b += J.bpart[(int64_t)z * J.bstride + n];
      __syncthreads();
      sbr[tid] = b;
      __syncthreads();
      for (int h = 128; h > 0; h >>= 1) {
        if (tid < h) sbr[tid] += sbr[tid + h];
        __syncthreads();
      }
      const float sb = sbr[0];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int64_t i = i4 + k;
        if (on && zg == 0 && (int)(i / J.fK) == n) {
          const int kk = (int)(i - (int64_t)n * J.fK);
          tv[k] = fmaf(tv[k], J.fg[kk], sb * J.fb[kk]);
        }
      }
    }
  }
  if (on && zg == 0) {
    float4* out = reinterpret_cast<float4*>(J.out + i4);
    float4 r = make_float4(tv[0], tv[1], tv[2], tv[3]);
    if (a.accumulate) r = add4(*out, r);
    *out = r;
  }
}

}  // namespace

hipError_t launch_reduce_list(ReduceList& l, int accumulate, hipStream_t s) {
  if (l.over) return hipErrorInvalidValue;
  ReduceArgs a;
  uint32_t blk = 0;
  for (int i = 0; i < l.n; ++i) {
    ReduceJob& J = l.j[i];
    if (J.Z <= 0 || J.count <= 0) continue;
    // wide rows while the job's own workgroups fill the chip, or its chains are short anyway
    const int64_t wide = (J.count + 127) / 128;
    J.og = wide >= 512 || J.Z <= 64 ? 32 : (J.Z <= 1024 ? 8 : 2);
    J.blk0 = blk;
    blk += (uint32_t)((J.count + 4 * J.og - 1) / (4 * J.og));
  }
  // jobs without partials or outputs are dropped
  int n = 0;
  for (int i = 0; i < l.n; ++i)
    if (l.j[i].Z > 0 && l.j[i].count > 0) a.j[n++] = l.j[i];
  if (n == 0) return hipSuccess;
  a.n = n;
  a.accumulate = accumulate;
  k_reduce_list<<<blk, 256, 0, s>>>(a);
  return hipGetLastError();
}

}  // namespace tfm
