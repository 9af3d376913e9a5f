// Kernels of the float32 mode (and of bfloat16 shapes outside the bf16 matrix-core envelope):
// float32 arithmetic throughout, storage type T (float or bf16), products on the fp32 matrix
// cores (v_mfma_f32_16x16x4_f32).
#pragma once

#include "common.h"
#include "fast.h"

namespace tfm {

// Chunks of cells that the weight gradients of one backward pass are split into: Z chunks of
// `chunk` cells (a multiple of 32).  Z never falls as N grows, so the buffers sized for Nmax
// cells hold the partials of any N <= Nmax.
struct F32Split {
  int Z;
  int64_t chunk;
};
F32Split f32_split(int64_t N, int E, int H);
// Partial rows of one LayerNorm backward.
int f32_ln_rows(int64_t N);
// Floats of the weight and bias partials (all six products) and of the norm partials.
size_t f32_wpart_floats(int64_t Nmax, int E, int H);
size_t f32_lnpart_floats(int64_t Nmax, int E);

// One weight gradient: part[z][n][k] = sum over the cells m of chunk z of Y[m][n] X[m][k] and
// bpart[z][n] = sum of Y[m][n].  Y: compact rows, or ROWS_ITEM_HM (Y, Y2, Y3 the head-major item
// dQ, dK, dV); X: compact or native rows.
template <class T>
struct F32WgradJob {
  const T *Y, *Y2, *Y3, *X;
  float *part, *bpart;
  int32_t N, K, ymode, xmode;
  int32_t tile0, ntn;  // first tile of the job, tiles along N (set by the launch)
};
constexpr int F32_WGRADS = 6;
template <class T>
struct F32WgradArgs {
  F32WgradJob<T> j[F32_WGRADS];
  int32_t n, tiles, Z;
  int64_t M, chunk;
  Geo g;
};
// All weight gradients of one backward pass in one launch (a.j[0..n) filled in).
template <class T>
hipError_t launch_f32_wgrads(F32WgradArgs<T>& a, const F32Split& sp, hipStream_t s);

// h = LN(a + b), a in amode rows (compact or native), h in hmode rows; xhat, rstd compact.
template <class T>
hipError_t launch_f32_add_ln(const Geo& g, const T* a, int amode, const T* b, const float* gamma,
                             const float* beta, T* h, int hmode, T* xhat, float* rstd,
                             hipStream_t s);
// du = LN'(dy), dy = dya (amode rows) + dyb (compact, may be null); part [f32_ln_rows(N)][2E]
// receives per-workgroup column sums of dy xhat and dy.
template <class T>
hipError_t launch_f32_ln_bwd(const Geo& g, const T* dya, int amode, const T* dyb, const T* xhat,
                             const float* rstd, const float* gamma, T* du, float* part,
                             hipStream_t s);

// out[m][n] = sum_k A[m][k] W(n, k) with an epilogue; W(n, k) = W[n * K + k], or W[k * N + n] with
// wt (the transposed product of a backward pass).
enum {
  F32_BIAS = 0,      // out = acc (+ bias), compact
  F32_GELU = 1,      // out = acc + bias, out2 = GELU(out)
  F32_GELU_BWD = 2,  // out = acc * GELU'(aux)
  F32_ITEM_QKV = 3,  // acc + bias head-major into out, out2, out3 (K and V at train rows only)
  F32_DX = 4         // out (native rows) = acc + aux
};
template <class T>
struct F32LinArgs {
  int64_t M;
  int32_t N, K, amode, wt, epi;
  const T *A, *A2, *A3;  // rows of K values: compact, native, or ROWS_ITEM_HM (dQ, dK, dV)
  const float *W, *bias;
  const T* aux;          // compact [M][N]
  T *out, *out2, *out3;
  Geo g;
};
template <class T>
hipError_t launch_f32_linear(const F32LinArgs<T>& a, hipStream_t s);

// Item-axis attention (layouts as in attn.h), keys the first n_train rows of the column.  The
// backward writes dq, dk, dv head-major (dk, dv at train rows only); Dbuf [NC * heads * R] is
// scratch.  On both axes lse is the base-2 log-sum-exp of the scores times log2(e), written and read
// by these kernels only.
template <class T>
hipError_t launch_f32_item_fwd(const Geo& g, const T* q, const T* k, const T* v, T* o, float* lse,
                               hipStream_t s);
template <class T>
hipError_t launch_f32_item_bwd(const Geo& g, const T* q, const T* k, const T* v, const T* o,
                               const T* dout, const float* lse, float* Dbuf, T* dq, T* dk, T* dv,
                               hipStream_t s);

// Feature-axis attention over the active cells of a row (at most 256), layouts as in attn.h.
template <class T>
hipError_t launch_f32_feat_fwd(const Geo& g, const T* qkv, T* o, float* lse, hipStream_t s);
template <class T>
hipError_t launch_f32_feat_bwd(const Geo& g, const T* qkv, const T* o, const T* dout,
                               const float* lse, T* dqkv, hipStream_t s);

}  // namespace tfm
