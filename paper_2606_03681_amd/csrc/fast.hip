// Small kernels of the MFMA path: zero fill, the norms at the ends of a block, thinking rows.
#include "fast.h"
#include "mfma.h"

namespace tfm {

WOff weight_offsets(int E, int H) {
  WOff o;
  int64_t x = 0;
  o.qkv_f = x; x += 3LL * E * E;
  o.o_f = x; x += (int64_t)E * E;
  o.qkv_i = x; x += 3LL * E * E;
  o.o_i = x; x += (int64_t)E * E;
  o.w1 = x; x += (int64_t)H * E;
  o.w2 = x; x += (int64_t)E * H;
  o.fb = (x + 7) / 8 * 8; x = o.fb + 2 * (3LL * E + H);
  // the forward and the backward stream of the fused MLP share one region
  int64_t msz = 0;
  if (mlp_fused_ok(E, H))
    msz = mlp_fwd_stream_elems(E, H) > mlp_bwd_stream_elems(E, H) ? mlp_fwd_stream_elems(E, H)
                                                                   : mlp_bwd_stream_elems(E, H);
  o.ms = (x + 127) / 128 * 128; x = o.ms + msz;
  o.total = x;
  return o;
}

// One wave per native row (b, r): the row's S cells are S * per contiguous 16-byte pieces,
// written with consecutive lanes on consecutive pieces, zero where the piece's cell is
// inactive.  Rows of datasets with every cell active leave at once.
__global__ void k_zero_inactive(Geo g, uint4* __restrict__ x, int per) {
  const int64_t row = (int64_t)blockIdx.x * 4 + wave_id();
  if (row >= (int64_t)g.B * g.R) return;
  const int b = (int)(row / g.R);
  if (g.ds[b].S == g.S) return;
  const int lane = threadIdx.x & 63;
  const int32_t* cm = g.colmap + (int64_t)b * g.S;
  uint4* p = x + row * g.S * per;
  const uint4 z = make_uint4(0, 0, 0, 0);
  for (int i = lane; i < g.S * per; i += 64)
    if (cm[i / per] < 0) p[i] = z;
}

hipError_t launch_zero_inactive(const Geo& g, void* native, size_t elt, hipStream_t s) {
  const int64_t rows = (int64_t)g.B * g.R;
  k_zero_inactive<<<(unsigned)((rows + 3) / 4), 256, 0, s>>>(
      g, reinterpret_cast<uint4*>(native), (int)(g.E * elt / 16));
  return hipGetLastError();
}

// LN3 backward from the native dY: 512 threads = 16 half-waves; a half-wave owns one cell at a
// time, lane l holding features 8l .. 8l+7 (E <= 256) in 16-byte pieces.  A block covers
// LN_CELLS consecutive compact cells; half-wave h takes cells h, h + 16, ..., four per batch
// with all their loads in flight, and keeps running column sums of dY * xhat and dY.
// LN_CELLS is 256 where that many cells a block still fill the chip, else 64 (one batch a
// half-wave): at 21,000 cells 82 blocks of 256 left two thirds of the CUs idle (22 us).
constexpr int LN_BATCH = 4;
static int ln_cells(int64_t N) { return N >= 256 * 1024 ? 256 : 64; }

template <int LN_CELLS>
__global__ __launch_bounds__(512) void k_ln_out_bwd(Geo g, const bf16* __restrict__ dY,
                                                    const bf16* __restrict__ xhat,
                                                    const float* __restrict__ rstd,
                                                    const float* __restrict__ gamma,
                                                    bf16* __restrict__ dz,
                                                    float* __restrict__ part) {
  __shared__ float red[16][2][256];
  const int tid = threadIdx.x, hw = tid >> 5, l = tid & 31;
  const int E = g.E;
  const bool act = 8 * l < E;
  float gm[8], cs1[8], cs2[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    gm[j] = act ? gamma[8 * l + j] : 0.f;
    cs1[j] = cs2[j] = 0.f;
  }
  const int64_t c0 = (int64_t)blockIdx.x * LN_CELLS;
  const int col0 = (int)(c0 / g.R), r0 = (int)(c0 - (int64_t)col0 * g.R);
  for (int base = hw; base < LN_CELLS; base += 16 * LN_BATCH) {
    uint4 dyv[LN_BATCH], xv[LN_BATCH];
    float rs[LN_BATCH];
    int64_t pc[LN_BATCH];
    bool ok[LN_BATCH];
#pragma unroll
    for (int u = 0; u < LN_BATCH; ++u) {
      const int cc = base + 16 * u;
      const int64_t p = c0 + cc;
      pc[u] = p;
      ok[u] = cc < LN_CELLS && p < g.N;
      dyv[u] = xv[u] = make_uint4(0, 0, 0, 0);
      rs[u] = 0.f;
      if (ok[u]) {
        int col = col0, r = r0 + cc;
        while (r >= g.R) {
          r -= g.R;
          ++col;
        }
        const int64_t nat = g.col_cell0[col] + (int64_t)r * g.S;
        rs[u] = rstd[p];
        if (act) {
          dyv[u] = ldu4(dY + nat * E + 8 * l);
          xv[u] = ldu4(xhat + p * E + 8 * l);
        }
      }
    }
#pragma unroll
    for (int u = 0; u < LN_BATCH; ++u) {
      float dy[8], x[8];
      float s1 = 0.f, s2 = 0.f;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        dy[j] = bf2f(u4_elem(dyv[u], j));
        x[j] = bf2f(u4_elem(xv[u], j));
        cs1[j] += dy[j] * x[j];
        cs2[j] += dy[j];
        s1 += dy[j] * gm[j];
        s2 += dy[j] * gm[j] * x[j];
      }
      s1 = half32_sum(s1);
      s2 = half32_sum(s2);
      const float m1 = s1 / E, m2 = s2 / E;
      if (ok[u] && act) {
        uint4 o;
        o.x = pack2(rs[u] * (dy[0] * gm[0] - m1 - x[0] * m2), rs[u] * (dy[1] * gm[1] - m1 - x[1] * m2));
        o.y = pack2(rs[u] * (dy[2] * gm[2] - m1 - x[2] * m2), rs[u] * (dy[3] * gm[3] - m1 - x[3] * m2));
        o.z = pack2(rs[u] * (dy[4] * gm[4] - m1 - x[4] * m2), rs[u] * (dy[5] * gm[5] - m1 - x[5] * m2));
        o.w = pack2(rs[u] * (dy[6] * gm[6] - m1 - x[6] * m2), rs[u] * (dy[7] * gm[7] - m1 - x[7] * m2));
        stu4(dz + pc[u] * E + 8 * l, o);
      }
    }
  }
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    red[hw][0][8 * l + j] = cs1[j];
    red[hw][1][8 * l + j] = cs2[j];
  }
  __syncthreads();
  if (tid < 2 * E) {
    const int t = tid / E, e = tid % E;
    float sm = 0.f;
#pragma unroll
    for (int h = 0; h < 16; ++h) sm += red[h][t][e];
    part[(int64_t)blockIdx.x * 2 * E + t * E + e] = sm;
  }
}

hipError_t launch_ln_out_bwd(const Geo& g, const bf16* dY, const bf16* xhat, const float* rstd,
                             const float* gamma, bf16* dz, float* part, int* nblocks,
                             hipStream_t s) {
  const int cells = ln_cells(g.N);
  const unsigned nb = (unsigned)((g.N + cells - 1) / cells);
  *nblocks = (int)nb;
  if (cells == 64) k_ln_out_bwd<64><<<nb, 512, 0, s>>>(g, dY, xhat, rstd, gamma, dz, part);
  else k_ln_out_bwd<256><<<nb, 512, 0, s>>>(g, dY, xhat, rstd, gamma, dz, part);
  return hipGetLastError();
}

// Pre-norm block input: x' = decay * X (native rows) and r = gamma x' / sqrt(mean(x'^2) + eps),
// both written compact, with rstd.  Same thread layout as the LN3 backward above: a half-wave
// per cell, lane l holding features 8l .. 8l+7, four cells per half-wave in flight.
template <int LN_CELLS>
__global__ __launch_bounds__(512) void k_rms_in(Geo g, const bf16* __restrict__ X, float decay,
                                                const float* __restrict__ gamma, float eps,
                                                bf16* __restrict__ xs, bf16* __restrict__ r,
                                                float* __restrict__ rstd) {
  const int tid = threadIdx.x, hw = tid >> 5, l = tid & 31;
  const int E = g.E;
  const bool act = 8 * l < E;
  float gm[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) gm[j] = act ? gamma[8 * l + j] : 0.f;
  const int64_t c0 = (int64_t)blockIdx.x * LN_CELLS;
  const int col0 = (int)(c0 / g.R), r0 = (int)(c0 - (int64_t)col0 * g.R);
  for (int base = hw; base < LN_CELLS; base += 16 * LN_BATCH) {
    uint4 xv[LN_BATCH];
    int64_t pc[LN_BATCH];
    bool ok[LN_BATCH];
#pragma unroll
    for (int u = 0; u < LN_BATCH; ++u) {
      const int cc = base + 16 * u;
      const int64_t p = c0 + cc;
      pc[u] = p;
      ok[u] = cc < LN_CELLS && p < g.N;
      xv[u] = make_uint4(0, 0, 0, 0);
      if (ok[u] && act) {
        int col = col0, rr = r0 + cc;
        while (rr >= g.R) {
          rr -= g.R;
          ++col;
        }
        const int64_t nat = g.col_cell0[col] + (int64_t)rr * g.S;
        xv[u] = ldu4(X + nat * E + 8 * l);
      }
    }
#pragma unroll
    for (int u = 0; u < LN_BATCH; ++u) {
      float x[8];
      float ss = 0.f;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        x[j] = decay * bf2f(u4_elem(xv[u], j));
        ss += x[j] * x[j];
      }
      ss = half32_sum(ss);
      const float rs = 1.0f / sqrtf(ss / E + eps);
      if (ok[u] && l == 0) rstd[pc[u]] = rs;
      if (ok[u] && act) {
        uint4 a, b;
        a.x = pack2(x[0], x[1]); a.y = pack2(x[2], x[3]);
        a.z = pack2(x[4], x[5]); a.w = pack2(x[6], x[7]);
        b.x = pack2(gm[0] * x[0] * rs, gm[1] * x[1] * rs);
        b.y = pack2(gm[2] * x[2] * rs, gm[3] * x[3] * rs);
        b.z = pack2(gm[4] * x[4] * rs, gm[5] * x[5] * rs);
        b.w = pack2(gm[6] * x[6] * rs, gm[7] * x[7] * rs);
        stu4(xs + pc[u] * E + 8 * l, a);
        stu4(r + pc[u] * E + 8 * l, b);
      }
    }
  }
}

hipError_t launch_rms_in(const Geo& g, const bf16* X, float decay, const float* gamma, float eps,
                         bf16* xs, bf16* r, float* rstd, hipStream_t s) {
  const int cells = ln_cells(g.N);
  const unsigned nb = (unsigned)((g.N + cells - 1) / cells);
  if (nb == 0) return hipSuccess;
  if (cells == 64) k_rms_in<64><<<nb, 512, 0, s>>>(g, X, decay, gamma, eps, xs, r, rstd);
  else k_rms_in<256><<<nb, 512, 0, s>>>(g, X, decay, gamma, eps, xs, r, rstd);
  return hipGetLastError();
}

// Thinking rows: rows [0, T) of X get the table (float32 [T][E]) at active cell columns and 0 at
// inactive ones; elements [i0, i0 + threads) of those rows, one a thread.
template <class TT>
__global__ void k_thinking_fwd(Geo g, int T, const float* __restrict__ table, TT* __restrict__ X,
                               int64_t i0) {
  const int64_t i = i0 + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t per = (int64_t)T * g.S * g.E;
  if (i >= per * g.B) return;
  const int b = (int)(i / per);
  const int64_t rest = i - b * per;
  const int t = (int)(rest / ((int64_t)g.S * g.E));
  const int c = (int)(rest / g.E % g.S);
  const int e = (int)(rest % g.E);
  const bool act = g.colmap[b * g.S + c] >= 0;
  st(X + (((int64_t)b * g.R + t) * g.S + c) * g.E + e, act ? table[t * g.E + e] : 0.f);
}

// dtable[t][e] (+)= sum over datasets b and active columns c of dX[b][t][c][e], in (b, c) order.
template <class TT>
__global__ void k_thinking_bwd(Geo g, int T, const TT* __restrict__ dX, float* __restrict__ dtable,
                               int accumulate) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)T * g.E) return;
  const int t = (int)(i / g.E), e = (int)(i % g.E);
  float s = 0.f;
  for (int b = 0; b < g.B; ++b)
    for (int c = 0; c < g.S; ++c)
      if (g.colmap[b * g.S + c] >= 0) s += ld(dX + (((int64_t)b * g.R + t) * g.S + c) * g.E + e);
  dtable[i] = (accumulate ? dtable[i] : 0.f) + s;
}

template <class TT>
hipError_t launch_thinking_fwd(const Geo& g, int T, const float* table, TT* X, hipStream_t s) {
  const int64_t n = (int64_t)g.B * T * g.S * g.E;
  constexpr int64_t per = MAX_THREADS / 256 * 256;
  for (int64_t i = 0; i < n; i += per)
    k_thinking_fwd<TT><<<(unsigned)(((n - i < per ? n - i : per) + 255) / 256), 256, 0, s>>>(
        g, T, table, X, i);
  return hipGetLastError();
}

template <class TT>
hipError_t launch_thinking_bwd(const Geo& g, int T, const TT* dX, float* dtable, int accumulate,
                               hipStream_t s) {
  const int64_t n = (int64_t)T * g.E;
  if (n == 0) return hipSuccess;
  k_thinking_bwd<TT><<<(unsigned)((n + 255) / 256), 256, 0, s>>>(g, T, dX, dtable, accumulate);
  return hipGetLastError();
}

template hipError_t launch_thinking_fwd<float>(const Geo&, int, const float*, float*, hipStream_t);
template hipError_t launch_thinking_fwd<bf16>(const Geo&, int, const float*, bf16*, hipStream_t);
template hipError_t launch_thinking_bwd<float>(const Geo&, int, const float*, float*, int,
                                               hipStream_t);
template hipError_t launch_thinking_bwd<bf16>(const Geo&, int, const bf16*, float*, int,
                                              hipStream_t);

int64_t ln_part_floats(int64_t cells, int E) { return gemm_max_tiles(cells) * 2 * E; }

size_t fast_workspace_bytes(int64_t cells, int E, int H) {
  const WOff wo = weight_offsets(E, H);
  return 2 * (size_t)wo.total * 2 + 1024                   // w and wt
         + 3 * (size_t)ln_part_floats(cells, E) * 4 + 256  // norm-backward column partials
         + wgrad_part_floats(cells, E, H) * 4 + 256;       // weight and bias partials
}

}  // namespace tfm
