// Plan and weight preparation (declarations in setup.h).
//
// Workgroups take one kind of work each, by block range: columns of the plan, 2,048-element pieces
// of the weight copies, outputs of the folded biases, pieces of the fused MLP's weight stream.
// These were five launches of 4.5 to 7 us a call for a few hundred KB; on tables of a few
// thousand cells that was a quarter of a forward pass.
#include "setup.h"

#include "kernels.h"
#include "mfma.h"

namespace tfm {

namespace {

struct Plan {
  SetupPlan p;
  int32_t from_args;
  int32_t v[SETUP_BLOB];
};

// first block of each kind of work
struct Ranges {
  uint32_t w, wt, bias, stream, end;
};

__device__ __forceinline__ void expand_column(const Plan& P, int t) {
  const SetupPlan& p = P.p;
  if (t >= p.B * p.S) return;
  const int b = t / p.S, c = t - b * p.S;
  const int stride = 4 + p.words;
  const int32_t* e = P.from_args ? P.v + b * stride : p.dblob + b * stride;
  if (c == 0) p.ds[b] = DsInfo{e[0], e[1], e[2], 0};
  const uint32_t word = (uint32_t)e[4 + (c >> 5)];
  if (!((word >> (c & 31)) & 1u)) {
    p.colmap[t] = -1;
    return;
  }
  int k = __popc(word & ((1u << (c & 31)) - 1u));
  for (int w = 0; w < (c >> 5); ++w) k += __popc((uint32_t)e[4 + w]);
  const int col = e[1] + k;
  p.colmap[t] = col;
  p.col_cell0[col] = (int64_t)b * p.R * p.S + c;
  p.col_ntr[col] = e[0];
  p.cord[e[3] + k] = col;
}

struct Mats {
  int64_t src[6], dst[6];
  int rows[6], cols[6];
};
__device__ __forceinline__ Mats mats(int E, int H, const WOff& wo) {
  const int64_t E2 = (int64_t)E * E;
  return Mats{{0, 3 * E2 + 3 * E, 4 * E2 + 4 * E, 7 * E2 + 7 * E, 8 * E2 + 8 * E,
               8 * E2 + 8 * E + (int64_t)H * E + H},
              {wo.qkv_f, wo.o_f, wo.qkv_i, wo.o_i, wo.w1, wo.w2},
              {3 * E, E, 3 * E, E, H, E},
              {E, E, E, E, E, H}};
}

__device__ __forceinline__ uint4 pack8(const float* v) {
  return make_uint4(pack2(v[0], v[1]), pack2(v[2], v[3]), pack2(v[4], v[5]), pack2(v[6], v[7]));
}
__device__ __forceinline__ void ld8f(const float* p, float* v) {
  const float4 a = reinterpret_cast<const float4*>(p)[0], b = reinterpret_cast<const float4*>(p)[1];
  v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
  v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}

// Eight consecutive elements (t a multiple of 8) of the fused MLP's weight streams: fragments of
// 512 elements in lane order, lane (g, r) holding row r and eight k values (order described in
// mlp.hip: 8g .. 8g+7 for the item out-projection, 4g .. 4g+3 and 16+4g .. 16+4g+3 of each
// 32-wide block elsewhere).
__device__ __forceinline__ void ld_perm(const float* p, int g, float* v) {
  const float4 a = *reinterpret_cast<const float4*>(p + 4 * g);
  const float4 b = *reinterpret_cast<const float4*>(p + 16 + 4 * g);
  v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
  v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}
__device__ __forceinline__ int perm_k(int g, int j) { return j < 4 ? 4 * g + j : 12 + 4 * g + j; }

__device__ __forceinline__ void mlp_fwd_stream8(const float* wo, const float* w1, const float* g2,
                                                const float* w2, int E, int H, int64_t t,
                                                float* v) {
  const int NE = E / 16, NK = E / 32, FPS = 2 * NE;  // fragments per stage
  const int lane = (int)((t >> 3) & 63);
  const int64_t f = t >> 9;  // fragment index in the stream
  const int st = (int)(f / FPS), fi = (int)(f % FPS);
  const int g = lane >> 4, r = lane & 15;
  if (st < NK / 2) {  // Wo_i: rows = output features, k = input features (natural order)
    const int kk = fi / NE, eb = fi % NE;
    ld8f(wo + (int64_t)(eb * 16 + r) * E + (2 * st + kk) * 32 + 8 * g, v);
    return;
  }
  const int c = st - NK / 2;
  if (fi < 2 * NK) {  // W1' = W1 diag(g2): rows = hidden units, k = features (permuted)
    const int hb = fi / NK, ks = fi % NK;
    float gm[8];
    ld_perm(w1 + (int64_t)(c * 32 + hb * 16 + r) * E + ks * 32, g, v);
    ld_perm(g2 + ks * 32, g, gm);
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] *= gm[j];
  } else {  // W2: rows = output features, k = the chunk's hidden units (permuted)
    const int eb = fi - 2 * NK;
    ld_perm(w2 + (int64_t)(eb * 16 + r) * H + c * 32, g, v);
  }
}

__device__ __forceinline__ void mlp_bwd_stream8(const float* w1, const float* g2, const float* w2,
                                                int E, int H, int64_t t, float* v) {
  const int NE = E / 16, NK = E / 32, FPS = 4 * NK + NE;
  const int lane = (int)((t >> 3) & 63);
  const int64_t f = t >> 9;
  const int c = (int)(f / FPS), fi = (int)(f % FPS);
  const int g = lane >> 4, r = lane & 15;
  if (fi < 4 * NK) {
    const int part = fi / (2 * NK), hb = (fi % (2 * NK)) / NK, ks = fi % NK;
    const int u = c * 32 + hb * 16 + r;
    if (part == 0) {
      float gm[8];
      ld_perm(w1 + (int64_t)u * E + ks * 32, g, v);
      ld_perm(g2 + ks * 32, g, gm);
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] *= gm[j];
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = w2[(int64_t)(ks * 32 + perm_k(g, j)) * H + u];
    }
  } else {
    const int eb = fi - 4 * NK;
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = w1[(int64_t)(c * 32 + perm_k(g, j)) * E + eb * 16 + r];
  }
}

__global__ __launch_bounds__(256) void k_setup(Plan P, SetupWeights W, WOff wo, Ranges r) {
  const int tid = threadIdx.x;
  if (blockIdx.x < r.w) {
    expand_column(P, (int)(blockIdx.x * 256 + tid));
    return;
  }
  const Mats m = mats(W.E, W.H, wo);
  if (blockIdx.x < r.bias) {
    // pieces of 2,048 elements; every matrix is a whole number of them (E and H are multiples
    // of 64)
    const bool tr = blockIdx.x >= r.wt;
    uint32_t i = blockIdx.x - (tr ? r.wt : r.w);
    const uint32_t want = tr ? W.wt : W.w;
    int k = 0;
    for (; k < 6; ++k) {
      if (!((want >> k) & 1u)) continue;
      const uint32_t n = (uint32_t)((int64_t)m.rows[k] * m.cols[k] / 2048);
      if (i < n) break;
      i -= n;
    }
    float v[8];
    if (!tr) {
      const int64_t t = (int64_t)i * 2048 + 8 * tid;
      ld8f(W.params + m.src[k] + t, v);
      if (W.fold && (k == 2 || k == 4)) {
        // the fold scales input column c of Wqkv_i by g1[c] and of W1 by g2[c]
        const float* gm = (k == 2 ? W.f.g1 : W.f.g2) + t % m.cols[k];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] *= gm[j];
      }
      stu4(W.wout + m.dst[k] + t, pack8(v));
    } else {
      // 32 rows x 64 columns: reads along the rows, 16-byte writes along the transposed rows
      const int nc = m.cols[k] / 64;
      const int r0 = (int)(i / nc) * 32 + 8 * (tid >> 6), c = (int)(i % nc) * 64 + (tid & 63);
#pragma unroll
      for (int j = 0; j < 8; ++j)
        v[j] = W.params[m.src[k] + (int64_t)(r0 + j) * m.cols[k] + c];
      stu4(W.wtout + m.dst[k] + (int64_t)c * m.rows[k] + r0, pack8(v));
    }
    return;
  }
  const int E = W.E, H = W.H;
  if (blockIdx.x < r.stream) {
    // Folded biases, one wave per output: bqkv_i[n] + sum_k Wqkv_i[n][k] be1[k] for n < 3E, then
    // b1[m] + sum_k W1[m][k] be2[k]; float32, lane l summing k = l, l + 64, ... (a coalesced
    // read of the weight row), then the lanes' sums added in a fixed butterfly
    const int n = (int)(blockIdx.x - r.bias) * 4 + wave_id();
    if (n >= 3 * E + H) return;
    const int lane = tid & 63;
    const bool q = n < 3 * E;
    const float* row = W.params + (q ? m.src[2] + (int64_t)n * E : m.src[4] + (int64_t)(n - 3 * E) * E);
    const float* be = q ? W.f.be1 : W.f.be2;
    float acc = 0.f;
    for (int k = lane; k < E; k += 64) acc = fmaf(row[k], be[k], acc);
    acc = wave_reduce_sum(acc);
    if (lane == 0)
      reinterpret_cast<float*>(W.wout + wo.fb)[n] = (q ? W.f.bqkv_i[n] : W.f.b1[n - 3 * E]) + acc;
    return;
  }
  const int64_t t = ((int64_t)(blockIdx.x - r.stream) * 256 + tid) * 8;
  const float *wo_i = W.params + m.src[3], *w1 = W.params + m.src[4], *w2 = W.params + m.src[5];
  float v[8];
  if (W.stream == 1) {
    if (t >= mlp_fwd_stream_elems(E, H)) return;
    mlp_fwd_stream8(wo_i, w1, W.f.g2, w2, E, H, t, v);
  } else {
    if (t >= mlp_bwd_stream_elems(E, H)) return;
    mlp_bwd_stream8(w1, W.f.g2, w2, E, H, t, v);
  }
  stu4(W.wout + wo.ms + t, pack8(v));
}

}  // namespace

hipError_t launch_setup(const SetupPlan& p, const SetupWeights* w, hipStream_t s) {
  Plan P;
  P.p = p;
  const int64_t n = (int64_t)p.B * (4 + p.words);
  P.from_args = n <= SETUP_BLOB;
  if (P.from_args) {
    for (int64_t i = 0; i < n; ++i) P.v[i] = p.blob[i];
  } else {
    const hipError_t e = launch_upload(p.blob, n, p.dblob, s);
    if (e != hipSuccess) return e;
  }
  Ranges r;
  r.w = (uint32_t)(((int64_t)p.B * p.S + 255) / 256);
  r.wt = r.bias = r.stream = r.end = r.w;
  WOff wo{};
  if (w) {
    const int64_t E = w->E, H = w->H;
    if (E % 64 || H % 64) return hipErrorInvalidValue;
    wo = weight_offsets(w->E, w->H);
    const int64_t cells[6] = {3 * E * E, E * E, 3 * E * E, E * E, H * E, E * H};
    for (int k = 0; k < 6; ++k)
      if ((w->w >> k) & 1u) r.wt += (uint32_t)(cells[k] / 2048);
    r.bias = r.wt;
    for (int k = 0; k < 6; ++k)
      if ((w->wt >> k) & 1u) r.bias += (uint32_t)(cells[k] / 2048);
    r.stream = r.bias + (w->fold ? (uint32_t)((3 * E + H + 3) / 4) : 0);
    const int64_t ms = w->stream == 1 ? mlp_fwd_stream_elems(w->E, w->H)
                                      : (w->stream == 2 ? mlp_bwd_stream_elems(w->E, w->H) : 0);
    r.end = r.stream + (uint32_t)((ms + 2047) / 2048);
  }
  k_setup<<<r.end, 256, 0, s>>>(P, w ? *w : SetupWeights{}, wo, r);
  return hipGetLastError();
}

}  // namespace tfm
