// Kernels of the float32 mode (declarations in f32.h).
//
// Every product runs on the fp32 matrix cores (operand layout in f32_frag.h).
#include "f32.h"

#include <algorithm>

#include "f32_frag.h"
#include "gelu.h"

namespace tfm {

namespace {

// Native cell of active cell p (p < 2^26, so 32-bit division).
__device__ __forceinline__ int64_t native32(const Geo& g, int64_t p) {
  const uint32_t col = (uint32_t)p / (uint32_t)g.R;
  const uint32_t r = (uint32_t)p - col * (uint32_t)g.R;
  return g.col_cell0[col] + (int64_t)r * g.S;
}

// ---- weight gradients -------------------------------------------------------------------------
// Contraction over cells: a workgroup sums one chunk of cells into a TS x TS tile of one weight
// gradient, four waves of TS/2 x TS/2, 32 cells per step through two LDS buffers with the next
// step's rows already in flight.  TS is 96 where E is a multiple of it (24 instead of 16 products
// for every float read: 21,000 cells, E = 192, H = 768 in 340 instead of 379 us), else 64.
// Both operands are read as rows of features (the contraction index is the slow one), row stride
// TS + 4 floats: the four lane groups of a fragment read take cells 4 apart, 16 banks apart.  All products of a backward pass are one launch: on a table of
// a few thousand cells no single one of them has enough tiles to fill the chip.
constexpr int WM = 32;   // cells per step
int f32_tile(int E) { return E % 96 == 0 ? 96 : 64; }

template <class T>
__device__ __forceinline__ float4 wg_load(const Geo& g, const T* p0, const T* p1, const T* p2,
                                          int mode, int64_t m, int64_t me, int f, int width) {
  if (m >= me || f >= width) return zf4();
  if (mode == ROWS_COMPACT) return ld4(p0 + m * width + f);
  if (mode == ROWS_NATIVE) return ld4(p0 + native32(g, m) * width + f);
  const uint32_t col = (uint32_t)m / (uint32_t)g.R;
  const int r = (int)((uint32_t)m - col * (uint32_t)g.R);
  int part;
  const int64_t off = item_hm_offset(g, col, r, f, &part);
  if (off < 0) return zf4();
  return ld4((part == 0 ? p0 : (part == 1 ? p1 : p2)) + off);
}

template <class T, int TS>
__global__ __launch_bounds__(256) void k_f32_wgrads(F32WgradArgs<T> a) {
  constexpr int WLS = TS + 4, NB = TS / 32, CH = TS / 4, NI = WM * CH / 256;
  __shared__ __attribute__((aligned(16))) float Ys[2][WM * WLS];
  __shared__ __attribute__((aligned(16))) float Xs[2][WM * WLS];
  // the tiles of one chunk sit on one XCD next to each other: its rows come from memory once
  const int idx = (int)(blockIdx.x >> 3), xcd = (int)(blockIdx.x & 7);
  const int z = (idx / a.tiles) * 8 + xcd, tl = idx % a.tiles;
  const int64_t mb = (int64_t)z * a.chunk;
  if (z >= a.Z || mb >= a.M) return;
  const int64_t me = mb + a.chunk < a.M ? mb + a.chunk : a.M;
  int ji = 0;
  while (ji + 1 < a.n && tl >= a.j[ji + 1].tile0) ++ji;
  const F32WgradJob<T>& J = a.j[ji];
  const int t = tl - J.tile0;
  const int n0 = (t % J.ntn) * TS, k0 = (t / J.ntn) * TS;
  const int tid = threadIdx.x, lane = tid & 63, w = wave_id();
  const int lg = lane >> 4, c = lane & 15;
  const int wn = (w >> 1) * (TS / 2), wk = (w & 1) * (TS / 2);
  // staging: piece p of a step is 4 features from 4 (p % CH) of cell p / CH
  float4 y[NI], x[NI];
  auto gload = [&](int64_t m0) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int p = tid + 256 * i, f = 4 * (p % CH);
      const int64_t m = m0 + p / CH;
      y[i] = wg_load<T>(a.g, J.Y, J.Y2, J.Y3, J.ymode, m, me, n0 + f, J.N);
      x[i] = wg_load<T>(a.g, J.X, nullptr, nullptr, J.xmode, m, me, k0 + f, J.K);
    }
  };
  auto sstore = [&](int b) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int p = tid + 256 * i, at = (p / CH) * WLS + 4 * (p % CH);
      st4(&Ys[b][at], y[i]);
      st4(&Xs[b][at], x[i]);
    }
  };
  f32x4 acc[NB][NB];
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[i][j] = zero4();
  const bool bias = k0 == 0;  // this tile also sums its columns of Y, 8 cells a wave and step
  float bs[2] = {0.f, 0.f};  // columns lane and 64 + lane
  gload(mb);
  sstore(0);
  __syncthreads();
  int b = 0;
  for (int64_t m0 = mb; m0 < me; m0 += WM, b ^= 1) {
    const bool more = m0 + WM < me;
    if (more) gload(m0 + WM);
#pragma unroll
    for (int s = 0; s < WM / 4; ++s) {
      const int row = 4 * lg + (s & 3) + 16 * (s >> 2);
      float av[NB], bv[NB];
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        av[i] = Ys[b][row * WLS + wn + 16 * i + c];
        bv[i] = Xs[b][row * WLS + wk + 16 * i + c];
      }
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[i][j] = mfma32(av[i], bv[j], acc[i][j]);
    }
    if (bias) {
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        bs[0] += Ys[b][(8 * w + r) * WLS + lane];
        if (TS > 64 && lane < TS - 64) bs[1] += Ys[b][(8 * w + r) * WLS + 64 + lane];
      }
    }
    if (more) sstore(b ^ 1);
    __syncthreads();
  }
  float* out = J.part + (int64_t)z * J.N * J.K;
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int n = n0 + wn + 16 * i + 4 * lg;
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int k = k0 + wk + 16 * j;
      if (n >= J.N || k >= J.K) continue;
#pragma unroll
      for (int r = 0; r < 4; ++r) out[(int64_t)(n + r) * J.K + k + c] = acc[i][j][r];
    }
  }
  if (bias) {
    float* R = Ys[0];
    R[w * 128 + lane] = bs[0];
    R[w * 128 + 64 + lane] = bs[1];
    __syncthreads();
    if (tid < TS && n0 + tid < J.N)
      J.bpart[(int64_t)z * J.N + n0 + tid] =
          (R[tid] + R[128 + tid]) + (R[256 + tid] + R[384 + tid]);
  }
}

// ---- LayerNorm --------------------------------------------------------------------------------
// One wave per cell from cell p0 up, lane l holding features 4l .. 4l+3 (E <= 256) in 16-byte
// pieces.
template <class T>
__global__ __launch_bounds__(256) void k_f32_add_ln(Geo g, int64_t p0, const T* __restrict__ a,
                                                    int amode,
                                                    const T* __restrict__ b,
                                                    const float* __restrict__ gamma,
                                                    const float* __restrict__ beta,
                                                    T* __restrict__ h, int hmode,
                                                    T* __restrict__ xhat,
                                                    float* __restrict__ rstd) {
  const int lane = threadIdx.x & 63, E = g.E;
  const int64_t p = p0 + (int64_t)blockIdx.x * 4 + wave_id();
  if (p >= g.N) return;
  const bool act = 4 * lane < E;
  const int64_t nat = amode == ROWS_NATIVE || hmode == ROWS_NATIVE ? native32(g, p) : 0;
  float u[4] = {0.f, 0.f, 0.f, 0.f};
  float4 gm = zf4(), be = zf4();
  if (act) {
    const float4 va = ld4(a + (amode == ROWS_NATIVE ? nat : p) * E + 4 * lane);
    const float4 vb = ld4(b + p * E + 4 * lane);
    gm = ld4(gamma + 4 * lane);
    be = ld4(beta + 4 * lane);
    u[0] = va.x + vb.x; u[1] = va.y + vb.y; u[2] = va.z + vb.z; u[3] = va.w + vb.w;
  }
  const float mean = wave_reduce_sum((u[0] + u[1]) + (u[2] + u[3])) / E;
  float v = 0.f;
  if (act) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      u[i] -= mean;
      v = fmaf(u[i], u[i], v);
    }
  }
  const float rs = 1.0f / sqrtf(wave_reduce_sum(v) / E + 1e-5f);
  if (act) {
#pragma unroll
    for (int i = 0; i < 4; ++i) u[i] *= rs;
    st4(xhat + p * E + 4 * lane, make_float4(u[0], u[1], u[2], u[3]));
    st4(h + (hmode == ROWS_NATIVE ? nat : p) * E + 4 * lane,
        make_float4(fmaf(gm.x, u[0], be.x), fmaf(gm.y, u[1], be.y), fmaf(gm.z, u[2], be.z),
                    fmaf(gm.w, u[3], be.w)));
  }
  if (lane == 0) rstd[p] = rs;
}

// Every wave takes cells blockIdx.x * 4 + wave, then a grid further on, and keeps running column
// sums; the four waves' sums are added in order at the end.
template <class T>
__global__ __launch_bounds__(256) void k_f32_ln_bwd(Geo g, const T* __restrict__ dya, int amode,
                                                    const T* __restrict__ dyb,
                                                    const T* __restrict__ xhat,
                                                    const float* __restrict__ rstd,
                                                    const float* __restrict__ gamma,
                                                    T* __restrict__ du, float* __restrict__ part) {
  __shared__ float red[4][512];
  const int lane = threadIdx.x & 63, w = wave_id(), E = g.E;
  const bool act = 4 * lane < E;
  const float4 gm = act ? ld4(gamma + 4 * lane) : zf4();
  const float gv[4] = {gm.x, gm.y, gm.z, gm.w};
  float c1[4] = {0.f, 0.f, 0.f, 0.f}, c2[4] = {0.f, 0.f, 0.f, 0.f};
  for (int64_t p = (int64_t)blockIdx.x * 4 + w; p < g.N; p += (int64_t)gridDim.x * 4) {
    float dy[4] = {0.f, 0.f, 0.f, 0.f}, x[4] = {0.f, 0.f, 0.f, 0.f};
    const float rs = rstd[p];
    if (act) {
      const float4 a = ld4(dya + (amode == ROWS_NATIVE ? native32(g, p) : p) * E + 4 * lane);
      const float4 b = dyb ? ld4(dyb + p * E + 4 * lane) : zf4();
      const float4 xv = ld4(xhat + p * E + 4 * lane);
      dy[0] = a.x + b.x; dy[1] = a.y + b.y; dy[2] = a.z + b.z; dy[3] = a.w + b.w;
      x[0] = xv.x; x[1] = xv.y; x[2] = xv.z; x[3] = xv.w;
    }
    float s1 = 0.f, s2 = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      c1[i] = fmaf(dy[i], x[i], c1[i]);
      c2[i] += dy[i];
      s1 = fmaf(dy[i], gv[i], s1);
      s2 = fmaf(dy[i] * gv[i], x[i], s2);
    }
    const float m1 = wave_reduce_sum(s1) / E, m2 = wave_reduce_sum(s2) / E;
    if (act) {
      float o[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) o[i] = rs * (dy[i] * gv[i] - m1 - x[i] * m2);
      st4(du + p * E + 4 * lane, make_float4(o[0], o[1], o[2], o[3]));
    }
  }
  if (act) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      red[w][4 * lane + i] = c1[i];
      red[w][E + 4 * lane + i] = c2[i];
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < 2 * E; i += 256)
    part[(int64_t)blockIdx.x * 2 * E + i] = (red[0][i] + red[1][i]) + (red[2][i] + red[3][i]);
}

// ---- linear layers ----------------------------------------------------------------------------
// 64 cells x 64 features a workgroup, four waves of 32 x 32, 32 values of k a stage through two
// LDS buffers, the next stage's rows in flight.  The weights are the A operand, so a lane ends
// with 4 consecutive features of one cell and the epilogues move 16 bytes per lane.  The 16 x 4
// products of a stage take k = 4g + j from lane group g in product j, so a lane reads 4
// consecutive k of its row at once; LDS rows of 36 floats keep those 16-byte reads apart.  A
// transposed weight is staged as it lies ([k][n], rows of 68 floats) and read one float a lane.
constexpr int LK = 32, LSR = 36, LST = 68;

template <class T, int AM, bool WT, int EPI>
__global__ __launch_bounds__(256) void k_f32_linear(F32LinArgs<T> a) {
  constexpr int WSZ = WT ? LK * LST : 64 * LSR;
  __shared__ __attribute__((aligned(16))) float As[2][64 * LSR];
  __shared__ __attribute__((aligned(16))) float Ws[2][WSZ];
  const Geo& g = a.g;
  const int tid = threadIdx.x, lane = tid & 63, w = wave_id();
  const int lg = lane >> 4, c = lane & 15;
  const int ntn = (a.N + 63) / 64;
  const int64_t m0 = (int64_t)(blockIdx.x / ntn) * 64;
  const int n0 = (int)(blockIdx.x % ntn) * 64;
  const int wm = (w >> 1) * 32, wn = (w & 1) * 32;
  // staging of A (and of W as stored): 4 values from 4 sc of rows sr, sr + 32
  const int sc = tid & 7, sr = tid >> 3;
  int64_t arow[2];
  uint32_t acol[2];
  int ar[2], antr[2];
  bool aok[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int64_t m = m0 + sr + 32 * i;
    aok[i] = m < a.M;
    arow[i] = aok[i] ? m * a.K : 0;
    acol[i] = 0;
    ar[i] = antr[i] = 0;
    if (AM == ROWS_NATIVE && aok[i]) arow[i] = native32(g, m) * a.K;
    if (AM == ROWS_ITEM_HM && aok[i]) {
      acol[i] = (uint32_t)m / (uint32_t)g.R;
      ar[i] = (int)((uint32_t)m - acol[i] * (uint32_t)g.R);
      antr[i] = g.col_ntr[acol[i]];
    }
  }
  float4 av[2], wv[2];
  auto gload = [&](int k0) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int k = k0 + 4 * sc;
      av[i] = zf4();
      if (AM == ROWS_ITEM_HM) {
        const int part = k / g.E, within = k - part * g.E;
        const int head = within / g.d, j = within - head * g.d;
        if (aok[i] && (part == 0 || ar[i] < antr[i]))
          av[i] = ld4((part == 0 ? a.A : (part == 1 ? a.A2 : a.A3)) +
                      (((int64_t)acol[i] * g.heads + head) * g.R + ar[i]) * g.d + j);
      } else if (aok[i]) {
        av[i] = ld4(a.A + arow[i] + k);
      }
      wv[i] = zf4();
      if (WT) {  // rows k = tid / 16 (+ 16), features 4 (tid % 16)
        const int kk = k0 + (tid >> 4) + 16 * i, n = n0 + 4 * (tid & 15);
        if (n < a.N) wv[i] = ld4(a.W + (int64_t)kk * a.N + n);
      } else {
        const int n = n0 + sr + 32 * i;
        if (n < a.N) wv[i] = ld4(a.W + (int64_t)n * a.K + k);
      }
    }
  };
  auto sstore = [&](int b) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      st4(&As[b][(sr + 32 * i) * LSR + 4 * sc], av[i]);
      if (WT) st4(&Ws[b][((tid >> 4) + 16 * i) * LST + 4 * (tid & 15)], wv[i]);
      else st4(&Ws[b][(sr + 32 * i) * LSR + 4 * sc], wv[i]);
    }
  };
  f32x4 acc[2][2];  // [feature block][cell block]
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = zero4();
  gload(0);
  sstore(0);
  __syncthreads();
  int b = 0;
  for (int k0 = 0; k0 < a.K; k0 += LK, b ^= 1) {
    const bool more = k0 + LK < a.K;
    if (more) gload(k0 + LK);
#pragma unroll
    for (int q = 0; q < LK / 16; ++q) {
      float4 xf[2];
      float wf[2][4];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        xf[i] = ld4(&As[b][(wm + 16 * i + c) * LSR + 16 * q + 4 * lg]);
        if (WT) {
#pragma unroll
          for (int j = 0; j < 4; ++j)
            wf[i][j] = Ws[b][(16 * q + 4 * lg + j) * LST + wn + 16 * i + c];
        } else {
          const float4 t = ld4(&Ws[b][(wn + 16 * i + c) * LSR + 16 * q + 4 * lg]);
          wf[i][0] = t.x; wf[i][1] = t.y; wf[i][2] = t.z; wf[i][3] = t.w;
        }
      }
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int x = 0; x < 2; ++x) {
            const float xj = j == 0 ? xf[x].x : (j == 1 ? xf[x].y : (j == 2 ? xf[x].z : xf[x].w));
            acc[i][x] = mfma32(wf[i][j], xj, acc[i][x]);
          }
    }
    if (more) sstore(b ^ 1);
    __syncthreads();
  }
#pragma unroll
  for (int x = 0; x < 2; ++x) {
    const int64_t m = m0 + wm + 16 * x + c;
    if (m >= a.M) continue;
    uint32_t col = 0;
    int r = 0, ntr = 0;
    int64_t nat = 0;
    if (EPI == F32_ITEM_QKV) {
      col = (uint32_t)m / (uint32_t)g.R;
      r = (int)((uint32_t)m - col * (uint32_t)g.R);
      ntr = g.col_ntr[col];
    }
    if (EPI == F32_DX) nat = native32(g, m);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int n = n0 + wn + 16 * i + 4 * lg;
      if (n >= a.N) continue;
      float4 v = make_float4(acc[i][x][0], acc[i][x][1], acc[i][x][2], acc[i][x][3]);
      if (EPI != F32_GELU_BWD && EPI != F32_DX && a.bias) {
        const float4 bb = ld4(a.bias + n);
        v = make_float4(v.x + bb.x, v.y + bb.y, v.z + bb.z, v.w + bb.w);
      }
      if (EPI == F32_BIAS) {
        st4(a.out + m * a.N + n, v);
      } else if (EPI == F32_GELU) {
        st4(a.out + m * a.N + n, v);
        st4(a.out2 + m * a.N + n, make_float4(gelu_exact(v.x), gelu_exact(v.y), gelu_exact(v.z),
                                              gelu_exact(v.w)));
      } else if (EPI == F32_GELU_BWD) {
        const float4 p = ld4(a.aux + m * a.N + n);
        st4(a.out + m * a.N + n,
            make_float4(v.x * gelu_exact_grad(p.x), v.y * gelu_exact_grad(p.y),
                        v.z * gelu_exact_grad(p.z), v.w * gelu_exact_grad(p.w)));
      } else if (EPI == F32_ITEM_QKV) {
        const int part = n / g.E, within = n - part * g.E;
        const int head = within / g.d, j = within - head * g.d;
        if (part > 0 && r >= ntr) continue;
        T* base = part == 0 ? a.out : (part == 1 ? a.out2 : a.out3);
        st4(base + (((int64_t)col * g.heads + head) * g.R + r) * g.d + j, v);
      } else {
        const float4 p = ld4(a.aux + m * a.N + n);
        st4(a.out + nat * a.N + n, make_float4(v.x + p.x, v.y + p.y, v.z + p.z, v.w + p.w));
      }
    }
  }
}

int f32_tiles(int ts, int N, int K) { return ((N + ts - 1) / ts) * ((K + ts - 1) / ts); }
int f32_all_tiles(int E, int H) {
  const int ts = f32_tile(E);
  return 2 * (f32_tiles(ts, 3 * E, E) + f32_tiles(ts, E, E) + f32_tiles(ts, H, E));
}
// Chunks asked for; never falls as N grows.
int64_t f32_want(int64_t N, int E, int H) {
  // enough workgroups for the chip, at least 64 cells and at most 2,048 in a chunk: a chunk's
  // partial tile (written and read once) is then no more than its operands' traffic, and no chain
  // of sums is longer
  const int tiles = f32_all_tiles(E, H);
  const int64_t fill = (2048 + tiles - 1) / tiles;
  return std::max<int64_t>(
      1, std::min<int64_t>((N + 63) / 64, std::max<int64_t>(fill, (N + 2047) / 2048)));
}

}  // namespace

F32Split f32_split(int64_t N, int E, int H) {
  const int64_t Z = f32_want(N, E, H);
  const int64_t chunk = std::max<int64_t>(((N + Z - 1) / Z + WM - 1) / WM * WM, WM);
  return F32Split{(int)std::max<int64_t>((N + chunk - 1) / chunk, 1), chunk};
}

int f32_ln_rows(int64_t N) {
  return (int)std::max<int64_t>(1, std::min<int64_t>(1024, (N + 15) / 16));
}

size_t f32_wpart_floats(int64_t Nmax, int E, int H) {
  // chunk rounding may leave fewer chunks than asked for, never more
  return (size_t)f32_want(Nmax, E, H) *
         (8 * (size_t)E * E + 2 * (size_t)E * H + 9 * (size_t)E + H);
}

size_t f32_lnpart_floats(int64_t Nmax, int E) { return (size_t)f32_ln_rows(Nmax) * 2 * E * 3; }

template <class T>
hipError_t launch_f32_wgrads(F32WgradArgs<T>& a, const F32Split& sp, hipStream_t s) {
  if (a.n < 1 || a.n > F32_WGRADS) return hipErrorInvalidValue;
  a.M = a.g.N;
  a.Z = sp.Z;
  a.chunk = sp.chunk;
  a.tiles = 0;
  const int ts = f32_tile(a.g.E);
  for (int i = 0; i < a.n; ++i) {
    a.j[i].tile0 = a.tiles;
    a.j[i].ntn = (a.j[i].N + ts - 1) / ts;
    a.tiles += f32_tiles(ts, a.j[i].N, a.j[i].K);
  }
  const unsigned grid = (unsigned)((sp.Z + 7) / 8 * 8 * a.tiles);
  if (ts == 96) k_f32_wgrads<T, 96><<<grid, 256, 0, s>>>(a);
  else k_f32_wgrads<T, 64><<<grid, 256, 0, s>>>(a);
  return hipGetLastError();
}

template <class T>
hipError_t launch_f32_add_ln(const Geo& g, const T* a, int amode, const T* b, const float* gamma,
                             const float* beta, T* h, int hmode, T* xhat, float* rstd,
                             hipStream_t s) {
  constexpr int64_t per = MAX_THREADS / 256;  // workgroups of one launch
  const int64_t nb = (g.N + 3) / 4;
  for (int64_t b0 = 0; b0 < nb; b0 += per)
    k_f32_add_ln<T><<<(unsigned)std::min(nb - b0, per), 256, 0, s>>>(
        g, 4 * b0, a, amode, b, gamma, beta, h, hmode, xhat, rstd);
  return hipGetLastError();
}

template <class T>
hipError_t launch_f32_ln_bwd(const Geo& g, const T* dya, int amode, const T* dyb, const T* xhat,
                             const float* rstd, const float* gamma, T* du, float* part,
                             hipStream_t s) {
  if (g.N <= 0) return hipSuccess;
  k_f32_ln_bwd<T><<<f32_ln_rows(g.N), 256, 0, s>>>(g, dya, amode, dyb, xhat, rstd, gamma, du,
                                                   part);
  return hipGetLastError();
}

template <class T>
hipError_t launch_f32_linear(const F32LinArgs<T>& a, hipStream_t s) {
  if (a.M <= 0) return hipSuccess;
  if (a.K % LK || a.N % 16) return hipErrorInvalidValue;
  const unsigned grid = (unsigned)((a.M + 63) / 64 * ((a.N + 63) / 64));
#define RUN(AM, WT, EPI) k_f32_linear<T, AM, WT, EPI><<<grid, 256, 0, s>>>(a)
  const int form = (a.wt ? 100 : 0) + a.amode * 10 + a.epi;
  switch (form) {
    case ROWS_NATIVE * 10 + F32_BIAS: RUN(ROWS_NATIVE, false, F32_BIAS); break;
    case ROWS_COMPACT * 10 + F32_BIAS: RUN(ROWS_COMPACT, false, F32_BIAS); break;
    case ROWS_COMPACT * 10 + F32_GELU: RUN(ROWS_COMPACT, false, F32_GELU); break;
    case ROWS_COMPACT * 10 + F32_ITEM_QKV: RUN(ROWS_COMPACT, false, F32_ITEM_QKV); break;
    case 100 + ROWS_COMPACT * 10 + F32_BIAS: RUN(ROWS_COMPACT, true, F32_BIAS); break;
    case 100 + ROWS_COMPACT * 10 + F32_GELU_BWD: RUN(ROWS_COMPACT, true, F32_GELU_BWD); break;
    case 100 + ROWS_COMPACT * 10 + F32_DX: RUN(ROWS_COMPACT, true, F32_DX); break;
    case 100 + ROWS_ITEM_HM * 10 + F32_BIAS: RUN(ROWS_ITEM_HM, true, F32_BIAS); break;
    default: return hipErrorInvalidValue;
  }
#undef RUN
  return hipGetLastError();
}

#define INST(T)                                                                               \
  template hipError_t launch_f32_wgrads<T>(F32WgradArgs<T>&, const F32Split&, hipStream_t);   \
  template hipError_t launch_f32_linear<T>(const F32LinArgs<T>&, hipStream_t);                \
  template hipError_t launch_f32_add_ln<T>(const Geo&, const T*, int, const T*, const float*, \
                                           const float*, T*, int, T*, float*, hipStream_t);   \
  template hipError_t launch_f32_ln_bwd<T>(const Geo&, const T*, int, const T*, const T*,     \
                                           const float*, const float*, T*, float*, hipStream_t);
INST(float)
INST(bf16)

}  // namespace tfm
