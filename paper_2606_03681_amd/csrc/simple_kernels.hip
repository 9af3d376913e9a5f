// Straightforward HIP kernels of the layer: fp32 arithmetic on VALU, any storage type.
// They serve the float32 mode, whose 1e-4 parity needs true fp32 products, and they are the
// baseline that the MFMA kernels of the bfloat16 mode are measured against.
#include <math.h>

#include "kernels.h"

namespace tfm {

namespace {

inline unsigned grid_for(int64_t n, int per_block = TFM_BLOCK) {
  int64_t g = (n + per_block - 1) / per_block;
  if (g < 1) g = 1;
  return (unsigned)g;
}

__device__ __forceinline__ int64_t gtid() {
  return (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
}
__device__ __forceinline__ int64_t gstride() { return (int64_t)gridDim.x * blockDim.x; }

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

}  // namespace

// ============================================================================ metadata
struct UploadChunk {
  int32_t n, off;
  int32_t v[504];
};

__global__ void k_upload(UploadChunk c, int32_t* dst) {
  for (int i = threadIdx.x; i < c.n; i += blockDim.x) dst[c.off + i] = c.v[i];
}

hipError_t launch_upload(const int32_t* host, int64_t count, int32_t* dst, hipStream_t s) {
  for (int64_t o = 0; o < count; o += 504) {
    UploadChunk c;
    c.n = (int32_t)((count - o) < 504 ? (count - o) : 504);
    c.off = (int32_t)o;
    for (int i = 0; i < c.n; ++i) c.v[i] = host[o + i];
    k_upload<<<1, TFM_BLOCK, 0, s>>>(c, dst);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

__global__ void k_expand_meta(const int32_t* blob, int B, int R, int S, int W, DsInfo* ds,
                              int32_t* col_ds, int32_t* col_c, int32_t* colmap,
                              int64_t* col_cell0, int32_t* col_ntr) {
  int64_t t = gtid();
  if (t >= (int64_t)B * S) return;
  int b = (int)(t / S), c = (int)(t % S);
  const int32_t* e = blob + (int64_t)b * (3 + W);
  const uint32_t* bits = (const uint32_t*)(e + 3);
  if (c == 0) ds[b] = DsInfo{e[0], e[1], e[2], 0};
  bool on = (bits[c >> 5] >> (c & 31)) & 1u;
  if (!on) {
    colmap[t] = -1;
    return;
  }
  int k = 0;
  for (int w = 0; w < (c >> 5); ++w) k += __popc(bits[w]);
  k += __popc(bits[c >> 5] & ((1u << (c & 31)) - 1u));
  int gcol = e[1] + k;
  col_ds[gcol] = b;
  col_c[gcol] = c;
  colmap[t] = gcol;
  col_cell0[gcol] = (int64_t)b * R * S + c;
  col_ntr[gcol] = e[0];
}

hipError_t launch_expand_meta(const int32_t* blob, int B, int R, int S, int words, DsInfo* ds,
                              int32_t* col_ds, int32_t* col_c, int32_t* colmap,
                              int64_t* col_cell0, int32_t* col_ntr, hipStream_t s) {
  k_expand_meta<<<grid_for((int64_t)B * S), TFM_BLOCK, 0, s>>>(blob, B, R, S, words, ds, col_ds,
                                                                 col_c, colmap, col_cell0,
                                                                 col_ntr);
  return hipGetLastError();
}

// ============================================================================ column sums
template <class T>
__global__ void k_colsum(int64_t M, int Nj, const T* __restrict__ A, int64_t lda,
                         const T* __restrict__ B, int64_t ldb, int64_t chunk,
                         float* __restrict__ part) {
  int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= Nj) return;
  int64_t mb = (int64_t)blockIdx.y * chunk;
  int64_t me = (mb + chunk < M) ? mb + chunk : M;
  float acc = 0.f;
  for (int64_t m = mb; m < me; ++m) {
    float v = ld(A + m * lda + j);
    if (B) v *= ld(B + m * ldb + j);
    acc += v;
  }
  part[(int64_t)blockIdx.y * Nj + j] = acc;
}

template <class T>
hipError_t launch_colsum(int64_t M, int Nj, const T* A, int64_t lda, const T* B, int64_t ldb,
                         int64_t chunk, float* partial, hipStream_t s) {
  int64_t Z = (M + chunk - 1) / chunk;
  if (Z < 1) Z = 1;
  dim3 grid((unsigned)((Nj + 255) / 256), (unsigned)Z);
  k_colsum<T><<<grid, 256, 0, s>>>(M, Nj, A, lda, B, ldb, chunk, partial);
  return hipGetLastError();
}

// ============================================================================ feature attention
// One thread per (row, head, query cell).  The cells of row (b, r) are
// p = (col0[b] + k) * R + r; q/k/v of cell p sit at qkv[p*3E + {0, E, 2E} + head*d].
template <class T, int D>
__global__ __launch_bounds__(256) void k_feat_attn_fwd(Geo g, const T* __restrict__ qkv,
                                                       T* __restrict__ o,
                                                       float* __restrict__ lse) {
  int64_t t = gtid();
  int64_t total = (int64_t)g.B * g.R * g.heads * g.S;
  if (t >= total) return;
  const int kq = (int)(t % g.S);
  t /= g.S;
  const int head = (int)(t % g.heads);
  const int64_t rho = t / g.heads;
  const int b = (int)(rho / g.R), r = (int)(rho % g.R);
  const DsInfo di = g.ds[b];
  if (kq >= di.S) return;
  const int E = g.E, E3 = 3 * g.E;
  const float tau = 1.0f / sqrtf((float)D);
  const int64_t pq = (int64_t)(di.col0 + kq) * g.R + r;
  float qv[D];
#pragma unroll
  for (int j = 0; j < D; ++j) qv[j] = ld(qkv + pq * E3 + head * D + j) * tau;
  float mx = -INFINITY;
  for (int kk = 0; kk < di.S; ++kk) {
    const T* kp = qkv + ((int64_t)(di.col0 + kk) * g.R + r) * E3 + E + head * D;
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < D; ++j) s = fmaf(qv[j], ld(kp + j), s);
    mx = fmaxf(mx, s);
  }
  float acc[D];
#pragma unroll
  for (int j = 0; j < D; ++j) acc[j] = 0.f;
  float sum = 0.f;
  for (int kk = 0; kk < di.S; ++kk) {
    const T* kp = qkv + ((int64_t)(di.col0 + kk) * g.R + r) * E3 + E + head * D;
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < D; ++j) s = fmaf(qv[j], ld(kp + j), s);
    float p = expf(s - mx);
    sum += p;
    const T* vp = kp + E;
#pragma unroll
    for (int j = 0; j < D; ++j) acc[j] = fmaf(p, ld(vp + j), acc[j]);
  }
  const float inv = 1.0f / sum;
#pragma unroll
  for (int j = 0; j < D; ++j) st(o + pq * E + head * D + j, acc[j] * inv);
  lse[pq * g.heads + head] = mx + logf(sum);
}

template <class T>
hipError_t launch_feat_attn_fwd_simple(const Geo& g, const T* qkv, T* o, float* lse,
                                       hipStream_t s) {
  int64_t total = (int64_t)g.B * g.R * g.heads * g.S;
  if (g.d == 16)
    k_feat_attn_fwd<T, 16><<<grid_for(total), TFM_BLOCK, 0, s>>>(g, qkv, o, lse);
  else if (g.d == 32)
    k_feat_attn_fwd<T, 32><<<grid_for(total), TFM_BLOCK, 0, s>>>(g, qkv, o, lse);
  else
    k_feat_attn_fwd<T, 64><<<grid_for(total), TFM_BLOCK, 0, s>>>(g, qkv, o, lse);
  return hipGetLastError();
}

// One thread per (row, head, cell i): dQ_i as a query, dK_i and dV_i as a key.
template <class T, int D>
__global__ __launch_bounds__(256) void k_feat_attn_bwd(Geo g, const T* __restrict__ qkv,
                                                       const T* __restrict__ o,
                                                       const T* __restrict__ dout,
                                                       const float* __restrict__ lse,
                                                       T* __restrict__ dqkv) {
  int64_t t = gtid();
  int64_t total = (int64_t)g.B * g.R * g.heads * g.S;
  if (t >= total) return;
  const int ki = (int)(t % g.S);
  t /= g.S;
  const int head = (int)(t % g.heads);
  const int64_t rho = t / g.heads;
  const int b = (int)(rho / g.R), r = (int)(rho % g.R);
  const DsInfo di = g.ds[b];
  if (ki >= di.S) return;
  const int E = g.E, E3 = 3 * g.E, hd = head * D;
  const float tau = 1.0f / sqrtf((float)D);
  const int64_t pi = (int64_t)(di.col0 + ki) * g.R + r;
  float qi[D], kv[D], vv[D], doi[D];
  float Di = 0.f;
#pragma unroll
  for (int j = 0; j < D; ++j) {
    qi[j] = ld(qkv + pi * E3 + hd + j);
    kv[j] = ld(qkv + pi * E3 + E + hd + j);
    vv[j] = ld(qkv + pi * E3 + 2 * E + hd + j);
    doi[j] = ld(dout + pi * E + hd + j);
    Di = fmaf(doi[j], ld(o + pi * E + hd + j), Di);
  }
  const float lsei = lse[pi * g.heads + head];
  float dq[D], dk[D], dv[D];
#pragma unroll
  for (int j = 0; j < D; ++j) dq[j] = dk[j] = dv[j] = 0.f;
  for (int kk = 0; kk < di.S; ++kk) {
    const int64_t pk = (int64_t)(di.col0 + kk) * g.R + r;
    const T* base = qkv + pk * E3 + hd;
    // cell i as the query, cell kk as the key
    float s = 0.f, dp = 0.f;
#pragma unroll
    for (int j = 0; j < D; ++j) {
      s = fmaf(qi[j], ld(base + E + j), s);
      dp = fmaf(doi[j], ld(base + 2 * E + j), dp);
    }
    float p = expf(s * tau - lsei);
    float ds = p * (dp - Di);
#pragma unroll
    for (int j = 0; j < D; ++j) dq[j] = fmaf(ds * tau, ld(base + E + j), dq[j]);
    // cell kk as the query, cell i as the key
    float s2 = 0.f, dp2 = 0.f, Dk = 0.f;
    const T* dok = dout + pk * E + hd;
    const T* ok = o + pk * E + hd;
#pragma unroll
    for (int j = 0; j < D; ++j) {
      float qk = ld(base + j);
      float dokj = ld(dok + j);
      s2 = fmaf(qk, kv[j], s2);
      dp2 = fmaf(dokj, vv[j], dp2);
      Dk = fmaf(dokj, ld(ok + j), Dk);
    }
    float p2 = expf(s2 * tau - lse[pk * g.heads + head]);
    float ds2 = p2 * (dp2 - Dk);
#pragma unroll
    for (int j = 0; j < D; ++j) {
      dk[j] = fmaf(ds2 * tau, ld(base + j), dk[j]);
      dv[j] = fmaf(p2, ld(dok + j), dv[j]);
    }
  }
#pragma unroll
  for (int j = 0; j < D; ++j) {
    st(dqkv + pi * E3 + hd + j, dq[j]);
    st(dqkv + pi * E3 + E + hd + j, dk[j]);
    st(dqkv + pi * E3 + 2 * E + hd + j, dv[j]);
  }
}

template <class T>
hipError_t launch_feat_attn_bwd_simple(const Geo& g, const T* qkv, const T* o, const T* dout,
                                       const float* lse, T* dqkv, hipStream_t s) {
  int64_t total = (int64_t)g.B * g.R * g.heads * g.S;
  if (g.d == 16)
    k_feat_attn_bwd<T, 16><<<grid_for(total), TFM_BLOCK, 0, s>>>(g, qkv, o, dout, lse, dqkv);
  else if (g.d == 32)
    k_feat_attn_bwd<T, 32><<<grid_for(total), TFM_BLOCK, 0, s>>>(g, qkv, o, dout, lse, dqkv);
  else
    k_feat_attn_bwd<T, 64><<<grid_for(total), TFM_BLOCK, 0, s>>>(g, qkv, o, dout, lse, dqkv);
  return hipGetLastError();
}

// ============================================================================ item attention
// One thread per (column, head, query row); keys are the train rows t < n_train.
template <class T, int D>
__global__ __launch_bounds__(256) void k_item_attn_fwd(Geo g, const T* __restrict__ q,
                                                       const T* __restrict__ k,
                                                       const T* __restrict__ v,
                                                       T* __restrict__ o,
                                                       float* __restrict__ lse) {
  int64_t t = gtid();
  if (t >= (int64_t)g.NC * g.heads * g.R) return;
  const int r = (int)(t % g.R);
  const int64_t ch = t / g.R;  // col * heads + head
  const int head = (int)(ch % g.heads);
  const int64_t col = ch / g.heads;
  const int n = g.col_ntr[col];
  const float tau = 1.0f / sqrtf((float)D);
  const int64_t base = ch * g.R;
  float qv[D];
#pragma unroll
  for (int j = 0; j < D; ++j) qv[j] = ld(q + (base + r) * D + j) * tau;
  float mx = -INFINITY;
  for (int tt = 0; tt < n; ++tt) {
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < D; ++j) s = fmaf(qv[j], ld(k + (base + tt) * D + j), s);
    mx = fmaxf(mx, s);
  }
  float acc[D];
#pragma unroll
  for (int j = 0; j < D; ++j) acc[j] = 0.f;
  float sum = 0.f;
  for (int tt = 0; tt < n; ++tt) {
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < D; ++j) s = fmaf(qv[j], ld(k + (base + tt) * D + j), s);
    float p = expf(s - mx);
    sum += p;
#pragma unroll
    for (int j = 0; j < D; ++j) acc[j] = fmaf(p, ld(v + (base + tt) * D + j), acc[j]);
  }
  const float inv = 1.0f / sum;
  const int64_t p = col * g.R + r;
#pragma unroll
  for (int j = 0; j < D; ++j) st(o + p * g.E + head * D + j, acc[j] * inv);
  lse[base + r] = mx + logf(sum);
}

template <class T>
hipError_t launch_item_attn_fwd_simple(const Geo& g, const T* q, const T* k, const T* v, T* o,
                                       float* lse, hipStream_t s) {
  int64_t total = (int64_t)g.NC * g.heads * g.R;
  if (g.d == 16)
    k_item_attn_fwd<T, 16><<<grid_for(total), TFM_BLOCK, 0, s>>>(g, q, k, v, o, lse);
  else if (g.d == 32)
    k_item_attn_fwd<T, 32><<<grid_for(total), TFM_BLOCK, 0, s>>>(g, q, k, v, o, lse);
  else
    k_item_attn_fwd<T, 64><<<grid_for(total), TFM_BLOCK, 0, s>>>(g, q, k, v, o, lse);
  return hipGetLastError();
}

template <class T, int D>
__global__ void k_item_rowdot(Geo g, const T* __restrict__ o, const T* __restrict__ dout,
                              float* __restrict__ Dv) {
  int64_t t = gtid();
  if (t >= (int64_t)g.NC * g.heads * g.R) return;
  const int r = (int)(t % g.R);
  const int64_t ch = t / g.R;
  const int head = (int)(ch % g.heads);
  const int64_t col = ch / g.heads;
  const int64_t p = (col * g.R + r) * g.E + head * D;
  float acc = 0.f;
#pragma unroll
  for (int j = 0; j < D; ++j) acc = fmaf(ld(o + p + j), ld(dout + p + j), acc);
  Dv[t] = acc;
}

template <class T, int D>
__global__ __launch_bounds__(256) void k_item_attn_dq(Geo g, const T* __restrict__ q,
                                                      const T* __restrict__ k,
                                                      const T* __restrict__ v,
                                                      const T* __restrict__ dout,
                                                      const float* __restrict__ lse,
                                                      const float* __restrict__ Dv,
                                                      T* __restrict__ dq) {
  int64_t t = gtid();
  if (t >= (int64_t)g.NC * g.heads * g.R) return;
  const int r = (int)(t % g.R);
  const int64_t ch = t / g.R;
  const int head = (int)(ch % g.heads);
  const int64_t col = ch / g.heads;
  const int n = g.col_ntr[col];
  const float tau = 1.0f / sqrtf((float)D);
  const int64_t base = ch * g.R;
  float qv[D], dov[D], acc[D];
  const int64_t p = (col * g.R + r) * g.E + head * D;
#pragma unroll
  for (int j = 0; j < D; ++j) {
    qv[j] = ld(q + (base + r) * D + j) * tau;
    dov[j] = ld(dout + p + j);
    acc[j] = 0.f;
  }
  const float L = lse[base + r], Dr = Dv[t];
  for (int tt = 0; tt < n; ++tt) {
    float s = 0.f, dp = 0.f;
#pragma unroll
    for (int j = 0; j < D; ++j) {
      s = fmaf(qv[j], ld(k + (base + tt) * D + j), s);
      dp = fmaf(dov[j], ld(v + (base + tt) * D + j), dp);
    }
    float ds = expf(s - L) * (dp - Dr) * tau;
#pragma unroll
    for (int j = 0; j < D; ++j) acc[j] = fmaf(ds, ld(k + (base + tt) * D + j), acc[j]);
  }
#pragma unroll
  for (int j = 0; j < D; ++j) st(dq + (base + r) * D + j, acc[j]);
}

template <class T, int D>
__global__ __launch_bounds__(256) void k_item_attn_dkv(Geo g, const T* __restrict__ q,
                                                       const T* __restrict__ k,
                                                       const T* __restrict__ v,
                                                       const T* __restrict__ dout,
                                                       const float* __restrict__ lse,
                                                       const float* __restrict__ Dv,
                                                       T* __restrict__ dk,
                                                       T* __restrict__ dv) {
  int64_t t = gtid();
  if (t >= (int64_t)g.NC * g.heads * g.R) return;
  const int tk = (int)(t % g.R);
  const int64_t ch = t / g.R;
  const int head = (int)(ch % g.heads);
  const int64_t col = ch / g.heads;
  const int n = g.col_ntr[col];
  if (tk >= n) return;
  const float tau = 1.0f / sqrtf((float)D);
  const int64_t base = ch * g.R;
  float kv[D], vv[D], ak[D], av[D];
#pragma unroll
  for (int j = 0; j < D; ++j) {
    kv[j] = ld(k + (base + tk) * D + j) * tau;
    vv[j] = ld(v + (base + tk) * D + j);
    ak[j] = av[j] = 0.f;
  }
  for (int r = 0; r < g.R; ++r) {
    const T* qr = q + (base + r) * D;
    const T* dor = dout + (col * g.R + r) * g.E + head * D;
    float s = 0.f, dp = 0.f;
#pragma unroll
    for (int j = 0; j < D; ++j) {
      s = fmaf(ld(qr + j), kv[j], s);
      dp = fmaf(ld(dor + j), vv[j], dp);
    }
    float p = expf(s - lse[base + r]);
    float ds = p * (dp - Dv[base + r]) * tau;
#pragma unroll
    for (int j = 0; j < D; ++j) {
      ak[j] = fmaf(ds, ld(qr + j), ak[j]);
      av[j] = fmaf(p, ld(dor + j), av[j]);
    }
  }
#pragma unroll
  for (int j = 0; j < D; ++j) {
    st(dk + (base + tk) * D + j, ak[j]);
    st(dv + (base + tk) * D + j, av[j]);
  }
}

template <class T>
hipError_t launch_item_attn_bwd_simple(const Geo& g, const T* q, const T* k, const T* v,
                                       const T* o, const T* dout, const float* lse, float* D,
                                       T* dq, T* dk, T* dv, hipStream_t s) {
  int64_t total = (int64_t)g.NC * g.heads * g.R;
  unsigned grid = grid_for(total);
  if (g.d == 16) {
    k_item_rowdot<T, 16><<<grid, TFM_BLOCK, 0, s>>>(g, o, dout, D);
    k_item_attn_dq<T, 16><<<grid, TFM_BLOCK, 0, s>>>(g, q, k, v, dout, lse, D, dq);
    k_item_attn_dkv<T, 16><<<grid, TFM_BLOCK, 0, s>>>(g, q, k, v, dout, lse, D, dk, dv);
  } else if (g.d == 32) {
    k_item_rowdot<T, 32><<<grid, TFM_BLOCK, 0, s>>>(g, o, dout, D);
    k_item_attn_dq<T, 32><<<grid, TFM_BLOCK, 0, s>>>(g, q, k, v, dout, lse, D, dq);
    k_item_attn_dkv<T, 32><<<grid, TFM_BLOCK, 0, s>>>(g, q, k, v, dout, lse, D, dk, dv);
  } else {
    k_item_rowdot<T, 64><<<grid, TFM_BLOCK, 0, s>>>(g, o, dout, D);
    k_item_attn_dq<T, 64><<<grid, TFM_BLOCK, 0, s>>>(g, q, k, v, dout, lse, D, dq);
    k_item_attn_dkv<T, 64><<<grid, TFM_BLOCK, 0, s>>>(g, q, k, v, dout, lse, D, dk, dv);
  }
  return hipGetLastError();
}

// ============================================================================ instantiations
#define INST(T)                                                                               \
  template hipError_t launch_colsum<T>(int64_t, int, const T*, int64_t, const T*, int64_t,   \
                                       int64_t, float*, hipStream_t);                        \
  template hipError_t launch_feat_attn_fwd_simple<T>(const Geo&, const T*, T*, float*,      \
                                                     hipStream_t);                           \
  template hipError_t launch_feat_attn_bwd_simple<T>(const Geo&, const T*, const T*,        \
                                                     const T*, const float*, T*,             \
                                                     hipStream_t);                           \
  template hipError_t launch_item_attn_fwd_simple<T>(const Geo&, const T*, const T*,        \
                                                     const T*, T*, float*, hipStream_t);     \
  template hipError_t launch_item_attn_bwd_simple<T>(const Geo&, const T*, const T*,        \
                                                     const T*, const T*, const T*,           \
                                                     const float*, float*, T*, T*, T*,       \
                                                     hipStream_t);

INST(float)
INST(bf16)

}  // namespace tfm
