// Internal declarations shared by the host library and the HIP kernels.
//
// Internal cell order.  Each dataset b keeps only its S_b active cell columns.  Active
// columns of all datasets are numbered globally, dataset-major.  Active cell p is (column
// g = p / R, row r = p % R), so every column is R consecutive cells — the item axis reads
// contiguous rows — and the cells of row (b, r) are p = (col0[b] + k) * R + r, k in [0, S_b).
//
// Item-axis Q/K/V are stored head-major per column: [g][head][R][d].
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tfm {

// Per-dataset metadata on the device.
struct DsInfo {
  int32_t n_train;  // train-prefix length
  int32_t col0;     // first global active column of the dataset
  int32_t S;        // number of active cell columns
  int32_t pad;
};

// Everything a kernel needs to map internal indices to the native [B][R][S][E] layout.
struct Geo {
  int32_t B, R, S, E, heads, d, H;
  int32_t NC;              // total active columns
  int64_t N;               // total active cells = NC * R
  const DsInfo* ds;        // [B]
  const int32_t* colmap;   // [B*S] native (b, c) -> global active column, or -1
  // Per active column: the native cell index of its row 0 (dataset b, cell column c: b R S + c)
  // and the train-prefix length of its dataset.
  const int64_t* col_cell0;  // [NC]
  const int32_t* col_ntr;    // [NC]
  int32_t nmax;              // longest train prefix over the datasets
};

// A subset of the active columns in a chosen order: column cols[i] for i < count; cols null
// means every column in order (count = NC).
struct ColList {
  const int32_t* cols;
  int32_t count;
};

// Threads of one launch: a grid of 2^32 or more is started modulo 2^32, without an error.  Kernels
// with a wave or a workgroup for each row or (column, head) problem reach that inside the supported
// envelope (many tables of a few rows or cells) and go in pieces, launches over some of the columns
// or datasets.
constexpr int64_t MAX_THREADS = (int64_t(1) << 32) - 1;

// fn(columns, c0) for successive pieces of the active columns: a Geo whose columns start at column
// c0 of g, of which per-column arrays (not cells of native tensors) are addressed from c0 on.
// threads: of one (column, head) problem; launches round their number up to a multiple of 8.
template <class F>
void by_columns(const Geo& g, int64_t threads, F fn) {
  const int64_t per = (MAX_THREADS / threads - 8) / g.heads;  // >= 1: R * E <= 715,827,882
  for (int64_t c0 = 0; c0 < g.NC; c0 += per) {
    Geo p = g;
    p.NC = (int32_t)(g.NC - c0 < per ? g.NC - c0 : per);
    p.N = (int64_t)p.NC * g.R;
    p.col_cell0 = g.col_cell0 + c0;
    p.col_ntr = g.col_ntr + c0;
    fn(p, c0);
  }
}
// fn(datasets) for successive pieces of the datasets: a Geo with some of them, whose columns and
// cells keep their numbers in g.  threads: of one row.
template <class F>
void by_datasets(const Geo& g, int64_t threads, F fn) {
  const int64_t per = (MAX_THREADS - 1024) / (threads * g.R);  // >= 1 as above
  for (int64_t b0 = 0; b0 < g.B; b0 += per) {
    Geo p = g;
    p.B = (int32_t)(g.B - b0 < per ? g.B - b0 : per);
    p.ds = g.ds + b0;
    fn(p);
  }
}

__host__ __device__ inline int64_t native_cell(const Geo& g, int64_t p) {
  int64_t col = p / g.R;
  int64_t r = p - col * g.R;
  return g.col_cell0[col] + r * g.S;
}

// bfloat16 storage as raw 16-bit patterns; round to nearest even on store.
typedef uint16_t bf16;

__device__ __forceinline__ float ld(const float* p) { return *p; }
__device__ __forceinline__ float ld(const bf16* p) {
  return __uint_as_float(((uint32_t)(*p)) << 16);
}
__device__ __forceinline__ void st(float* p, float v) { *p = v; }
__device__ __forceinline__ uint16_t f2bf(float v) {
  uint32_t u = __float_as_uint(v);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__device__ __forceinline__ void st(bf16* p, float v) { *p = f2bf(v); }

// Launch helpers return hipError_t of the launch.
#define TFM_BLOCK 256

}  // namespace tfm
