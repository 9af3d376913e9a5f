// Attention of the float32 mode (declarations in f32.h, operand layout in f32_frag.h): float32
// products on v_mfma_f32_16x16x4_f32, softmax in float32.
//
// A wave owns 16 queries (or, for the key and value gradients, 16 keys).  It computes score
// tiles with its own rows as the columns of the product (S^T = K Q^T; S = Q K^T for the key
// side), so that lane (g, c) holds four scores of its row c, at the other axis' rows
// 4g .. 4g+3: exactly the B operand of the next product when product r of four takes rows
// {r, 4 + r, 8 + r, 12 + r}.  Probabilities and score gradients therefore go from one product to
// the next in registers, and row sums and maxima are a register chain and two lane swaps.
// The former kernels gave each query one thread that walked every key, its row from L1 each
// time: 1.9, 1.0 and 1.7 ms for dQ, dK/dV and the forward of one 1,000 x 21 table.
#include <math.h>

#include "f32.h"
#include "f32_frag.h"

namespace tfm {

namespace {

__device__ __forceinline__ float el(const float4& v, int j) {
  return j == 0 ? v.x : (j == 1 ? v.y : (j == 2 ? v.z : v.w));
}
__device__ __forceinline__ float dot4(const float4& a, const float4& b) {
  return fmaf(a.x, b.x, fmaf(a.y, b.y, fmaf(a.z, b.z, a.w * b.w)));
}
// Queries are scaled by log2(e) / sqrt(d) as they are loaded, so that scores are exponents of 2 for
// v_exp_f32, and log-sum-exps are kept in base 2: every kernel forms a score from the same operands in
// the same order, so a dominant key's score less the log-sum-exp is exact, and its probability 1,
// however large the scores are.
constexpr float LOG2E = 1.4426950408889634f, LN2 = 0.69314718055994531f;
// What a running softmax subtracts from its scores at running maximum mx: 0 while every score was
// -infinity (a product that overflowed), whose terms are then 0 and not NaN, as they are to a later
// finite maximum.  A row of such scores alone ends as 0 / 0.
__device__ __forceinline__ float exp_ref(float mx) { return mx == -INFINITY ? 0.f : mx; }
__device__ __forceinline__ float4 scale4(const float4& a, float f) {
  return make_float4(a.x * f, a.y * f, a.z * f, a.w * f);
}

// Fragment of one row of D values: lane group g holds values 16 i + 4 g .. + 3 of it.
template <int D>
struct Row {
  float4 v[D / 16];
};
template <int D, class T>
__device__ __forceinline__ Row<D> ld_row(const T* p, bool ok, int lg) {
  Row<D> r;
#pragma unroll
  for (int i = 0; i < D / 16; ++i) r.v[i] = ok ? ld4(p + 16 * i + 4 * lg) : zf4();
  return r;
}
// 16 x 16 tile of row products: A's rows give the tile's rows, B's its columns.
template <int D>
__device__ __forceinline__ f32x4 rows_dot(const Row<D>& a, const Row<D>& b) {
  f32x4 acc = zero4();
#pragma unroll
  for (int i = 0; i < D / 16; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc = mfma32(el(a.v[i], j), el(b.v[i], j), acc);
  return acc;
}

// ---- item axis --------------------------------------------------------------------------------
// Workgroup: 64 rows of one (column, head) problem, 16 a wave, sharing 32-row tiles of the other
// axis through two LDS buffers (rows of D + 4 floats: both the 16-byte row reads and the 4-byte
// reads of four rows 4 apart are free of bank conflicts).  The workgroups of a problem run on
// one XCD.
constexpr int TK = 32;

struct Prob {
  int64_t ch, col;
  int head, blk;
  bool ok;
};
__device__ __forceinline__ Prob problem(const Geo& g, int nblk) {
  const int i = (int)(blockIdx.x >> 3), xcd = (int)(blockIdx.x & 7);
  Prob p;
  p.ch = (int64_t)(i / nblk) * 8 + xcd;
  p.blk = i % nblk;
  p.ok = p.ch < (int64_t)g.NC * g.heads;
  p.col = p.ch / g.heads;
  p.head = (int)(p.ch - p.col * g.heads);
  return p;
}

// Rows r0 .. r0 + 31 (below `rows`, else 0) of two row arrays: loaded to registers, then stored
// to a pair of LDS tiles.
template <class T, int D>
struct Stage {
  static constexpr int NI = (TK * D / 4 + 255) / 256;
  float4 a[NI], b[NI];
  __device__ __forceinline__ void load(const T* pa, int64_t lda, const T* pb, int64_t ldb, int r0,
                                       int rows) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int t = threadIdx.x + 256 * i, r = t / (D / 4), c4 = 4 * (t % (D / 4));
      const bool ok = t < TK * D / 4 && r0 + r < rows;
      a[i] = ok ? ld4(pa + (int64_t)(r0 + r) * lda + c4) : zf4();
      b[i] = ok ? ld4(pb + (int64_t)(r0 + r) * ldb + c4) : zf4();
    }
  }
  __device__ __forceinline__ void store(float* sa, float* sb) const {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int t = threadIdx.x + 256 * i, r = t / (D / 4), c4 = 4 * (t % (D / 4));
      if (t < TK * D / 4) {
        *reinterpret_cast<float4*>(&sa[r * (D + 4) + c4]) = a[i];
        *reinterpret_cast<float4*>(&sb[r * (D + 4) + c4]) = b[i];
      }
    }
  }
};

template <class T, int D>
__global__ __launch_bounds__(256) void k_f32_item_fwd(Geo g, const T* __restrict__ q,
                                                      const T* __restrict__ k,
                                                      const T* __restrict__ v,
                                                      T* __restrict__ o,
                                                      float* __restrict__ lse) {
  constexpr int LS = D + 4, NB = D / 16;
  __shared__ __attribute__((aligned(16))) float Ks[2][TK * LS];
  __shared__ __attribute__((aligned(16))) float Vs[2][TK * LS];
  const Prob P = problem(g, (g.R + 63) / 64);
  if (!P.ok) return;
  const int lane = threadIdx.x & 63, lg = lane >> 4, c = lane & 15;
  const int n = g.col_ntr[P.col], r = P.blk * 64 + 16 * wave_id() + c;
  const bool rok = r < g.R;
  const int64_t base = P.ch * g.R;
  const float tau = 1.0f / sqrtf((float)D);
  Row<D> qf = ld_row<D>(q + (base + r) * D, rok, lg);
#pragma unroll
  for (int i = 0; i < NB; ++i) qf.v[i] = scale4(qf.v[i], tau * LOG2E);
  f32x4 acc[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) acc[i] = zero4();
  float mx = -INFINITY, sum = 0.f;
  Stage<T, D> st;
  st.load(k + base * D, D, v + base * D, D, 0, n);
  st.store(Ks[0], Vs[0]);
  __syncthreads();
  int b = 0;
  for (int k0 = 0; k0 < n; k0 += TK, b ^= 1) {
    const bool more = k0 + TK < n;
    if (more) st.load(k + base * D, D, v + base * D, D, k0 + TK, n);
    f32x4 s[2];
    float tm = -INFINITY;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      s[kb] = rows_dot<D>(ld_row<D>(&Ks[b][(16 * kb + c) * LS], true, lg), qf);
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        if (k0 + 16 * kb + 4 * lg + x >= n) s[kb][x] = -INFINITY;
        tm = fmaxf(tm, s[kb][x]);
      }
    }
    const float mn = fmaxf(mx, rows4_max(tm)), ref = exp_ref(mn);
    const float al = exp2_hw(mx - ref);
    mx = mn;
    sum *= al;
#pragma unroll
    for (int i = 0; i < NB; ++i) acc[i] *= al;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        const float p = exp2_hw(s[kb][x] - ref);
        sum += p;
        const float* vr = &Vs[b][(16 * kb + 4 * lg + x) * LS + c];
#pragma unroll
        for (int i = 0; i < NB; ++i) acc[i] = mfma32(vr[16 * i], p, acc[i]);
      }
    if (more) st.store(Ks[b ^ 1], Vs[b ^ 1]);
    __syncthreads();
  }
  if (!rok) return;
  sum = rows4_sum(sum);
  const float inv = 1.0f / sum;
#pragma unroll
  for (int i = 0; i < NB; ++i)
    st4(o + (P.col * g.R + r) * g.E + P.head * D + 16 * i + 4 * lg, acc[i] * inv);
  if (lg == 0) lse[base + r] = mx + log2f(sum);
}

template <class T, int D>
__global__ __launch_bounds__(256) void k_f32_item_dq(Geo g, const T* __restrict__ q,
                                                     const T* __restrict__ k,
                                                     const T* __restrict__ v,
                                                     const T* __restrict__ o,
                                                     const T* __restrict__ dout,
                                                     const float* __restrict__ lse,
                                                     float* __restrict__ Dbuf,
                                                     T* __restrict__ dq) {
  constexpr int LS = D + 4, NB = D / 16;
  __shared__ __attribute__((aligned(16))) float Ks[2][TK * LS];
  __shared__ __attribute__((aligned(16))) float Vs[2][TK * LS];
  const Prob P = problem(g, (g.R + 63) / 64);
  if (!P.ok) return;
  const int lane = threadIdx.x & 63, lg = lane >> 4, c = lane & 15;
  const int n = g.col_ntr[P.col], r = P.blk * 64 + 16 * wave_id() + c;
  const bool rok = r < g.R;
  const int64_t base = P.ch * g.R, oc = (P.col * g.R + r) * g.E + P.head * D;
  const float tau = 1.0f / sqrtf((float)D);
  Row<D> qf = ld_row<D>(q + (base + r) * D, rok, lg);
  const Row<D> df = ld_row<D>(dout + oc, rok, lg), of = ld_row<D>(o + oc, rok, lg);
  float Dr = 0.f;
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    qf.v[i] = scale4(qf.v[i], tau * LOG2E);
    Dr += dot4(df.v[i], of.v[i]);
  }
  Dr = rows4_sum(Dr);
  const float L = rok ? lse[base + r] : 0.f;
  if (rok && lg == 0) Dbuf[base + r] = Dr;
  f32x4 acc[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) acc[i] = zero4();
  Stage<T, D> st;
  st.load(k + base * D, D, v + base * D, D, 0, n);
  st.store(Ks[0], Vs[0]);
  __syncthreads();
  int b = 0;
  for (int k0 = 0; k0 < n; k0 += TK, b ^= 1) {
    const bool more = k0 + TK < n;
    if (more) st.load(k + base * D, D, v + base * D, D, k0 + TK, n);
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      const f32x4 s = rows_dot<D>(ld_row<D>(&Ks[b][(16 * kb + c) * LS], true, lg), qf);
      const f32x4 dp = rows_dot<D>(ld_row<D>(&Vs[b][(16 * kb + c) * LS], true, lg), df);
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        const bool in = k0 + 16 * kb + 4 * lg + x < n;
        const float ds = in ? exp2_hw(s[x] - L) * (dp[x] - Dr) : 0.f;
        const float* kr = &Ks[b][(16 * kb + 4 * lg + x) * LS + c];
#pragma unroll
        for (int i = 0; i < NB; ++i) acc[i] = mfma32(kr[16 * i], ds, acc[i]);
      }
    }
    if (more) st.store(Ks[b ^ 1], Vs[b ^ 1]);
    __syncthreads();
  }
  if (!rok) return;
#pragma unroll
  for (int i = 0; i < NB; ++i) st4(dq + (base + r) * D + 16 * i + 4 * lg, acc[i] * tau);
}

template <class T, int D>
__global__ __launch_bounds__(256) void k_f32_item_dkv(Geo g, const T* __restrict__ q,
                                                      const T* __restrict__ k,
                                                      const T* __restrict__ v,
                                                      const T* __restrict__ dout,
                                                      const float* __restrict__ lse,
                                                      const float* __restrict__ Dbuf,
                                                      T* __restrict__ dk, T* __restrict__ dv) {
  constexpr int LS = D + 4, NB = D / 16;
  __shared__ __attribute__((aligned(16))) float Qs[2][TK * LS];
  __shared__ __attribute__((aligned(16))) float Os[2][TK * LS];
  __shared__ float Ls[2][TK], Ds[2][TK];
  const Prob P = problem(g, (g.nmax + 63) / 64);
  if (!P.ok) return;
  const int n = g.col_ntr[P.col];
  if (P.blk * 64 >= n) return;
  const int tid = threadIdx.x, lane = tid & 63, lg = lane >> 4, c = lane & 15;
  const int t = P.blk * 64 + 16 * wave_id() + c;
  const bool tok = t < n;
  const int64_t base = P.ch * g.R;
  const T* od = dout + P.col * g.R * g.E + P.head * D;
  const float tau = 1.0f / sqrtf((float)D);
  const Row<D> kf = ld_row<D>(k + (base + t) * D, tok, lg);
  const Row<D> vf = ld_row<D>(v + (base + t) * D, tok, lg);
  f32x4 ak[NB], av[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) ak[i] = av[i] = zero4();
  Stage<T, D> st;
  float sl = 0.f, sd = 0.f;
  auto load = [&](int r0) __attribute__((always_inline)) {
    st.load(q + base * D, D, od, g.E, r0, g.R);
    // rows past the end: zero dO, L and D give P = 1 against zero rows
    const bool ok = tid < TK && r0 + tid < g.R;
    sl = ok ? lse[base + r0 + tid] : 0.f;
    sd = ok ? Dbuf[base + r0 + tid] : 0.f;
  };
  auto store = [&](int b) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < st.NI; ++i) st.a[i] = scale4(st.a[i], tau * LOG2E);
    st.store(Qs[b], Os[b]);
    if (tid < TK) {
      Ls[b][tid] = sl;
      Ds[b][tid] = sd;
    }
  };
  load(0);
  store(0);
  __syncthreads();
  int b = 0;
  for (int r0 = 0; r0 < g.R; r0 += TK, b ^= 1) {
    const bool more = r0 + TK < g.R;
    if (more) load(r0 + TK);
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
      const f32x4 s = rows_dot<D>(ld_row<D>(&Qs[b][(16 * qb + c) * LS], true, lg), kf);
      const f32x4 dp = rows_dot<D>(ld_row<D>(&Os[b][(16 * qb + c) * LS], true, lg), vf);
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        const int row = 16 * qb + 4 * lg + x;
        const float p = exp2_hw(s[x] - Ls[b][row]);
        const float ds = p * (dp[x] - Ds[b][row]);
        const float* qr = &Qs[b][row * LS + c];
        const float* orow = &Os[b][row * LS + c];
#pragma unroll
        for (int i = 0; i < NB; ++i) {
          av[i] = mfma32(orow[16 * i], p, av[i]);
          ak[i] = mfma32(qr[16 * i], ds, ak[i]);
        }
      }
    }
    if (more) store(b ^ 1);
    __syncthreads();
  }
  if (!tok) return;
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    st4(dk + (base + t) * D + 16 * i + 4 * lg, ak[i] * LN2);  // Q carries tau log2(e)
    st4(dv + (base + t) * D + 16 * i + 4 * lg, av[i]);
  }
}

// ---- feature axis -----------------------------------------------------------------------------
// One wave per (row, head, 16 cells); the other cells' rows come straight from memory (a row's
// Q|K|V of one head are read by its at most 16 waves, which sit next to each other).
struct FeatTask {
  int S, r, head, b0;
  int64_t col0;
  bool ok;
};
__device__ __forceinline__ FeatTask feat_task(const Geo& g) {
  const int nblk = (g.S + 15) / 16;
  int64_t t = (int64_t)blockIdx.x * 4 + wave_id();
  FeatTask f;
  f.b0 = (int)(t % nblk) * 16;
  t /= nblk;
  f.head = (int)(t % g.heads);
  t /= g.heads;
  f.ok = t < (int64_t)g.B * g.R;
  if (!f.ok) return f;
  const int b = (int)(t / g.R);
  f.r = (int)(t - (int64_t)b * g.R);
  const DsInfo di = g.ds[b];
  f.S = di.S;
  f.col0 = di.col0;
  f.ok = f.b0 < f.S;
  return f;
}

template <class T, int D>
__global__ __launch_bounds__(256) void k_f32_feat_fwd(Geo g, const T* __restrict__ qkv,
                                                      T* __restrict__ o,
                                                      float* __restrict__ lse) {
  constexpr int NB = D / 16;
  const FeatTask F = feat_task(g);
  if (!F.ok) return;
  const int lane = threadIdx.x & 63, lg = lane >> 4, c = lane & 15;
  const int E = g.E, E3 = 3 * E, hd = F.head * D;
  auto cell = [&](int x) { return (F.col0 + x) * g.R + F.r; };
  const float tau = 1.0f / sqrtf((float)D);
  const int kq = F.b0 + c;
  const bool qok = kq < F.S;
  const int64_t pq = qok ? cell(kq) : 0;
  Row<D> qf = ld_row<D>(qkv + pq * E3 + hd, qok, lg);
#pragma unroll
  for (int i = 0; i < NB; ++i) qf.v[i] = scale4(qf.v[i], tau * LOG2E);
  f32x4 acc[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) acc[i] = zero4();
  float mx = -INFINITY, sum = 0.f;
  for (int k0 = 0; k0 < F.S; k0 += 16) {
    const bool kok = k0 + c < F.S;
    const Row<D> kf = ld_row<D>(qkv + (kok ? cell(k0 + c) : 0) * E3 + E + hd, kok, lg);
    float vv[4][NB];
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      const int kk = k0 + 4 * lg + x;
      const bool ok = kk < F.S;
      const T* vp = qkv + (ok ? cell(kk) : 0) * E3 + 2 * E + hd + c;
#pragma unroll
      for (int i = 0; i < NB; ++i) vv[x][i] = ok ? ld(vp + 16 * i) : 0.f;
    }
    f32x4 s = rows_dot<D>(kf, qf);
    float tm = -INFINITY;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      if (k0 + 4 * lg + x >= F.S) s[x] = -INFINITY;
      tm = fmaxf(tm, s[x]);
    }
    const float mn = fmaxf(mx, rows4_max(tm)), ref = exp_ref(mn);
    const float al = exp2_hw(mx - ref);
    mx = mn;
    sum *= al;
#pragma unroll
    for (int i = 0; i < NB; ++i) acc[i] *= al;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      const float p = exp2_hw(s[x] - ref);
      sum += p;
#pragma unroll
      for (int i = 0; i < NB; ++i) acc[i] = mfma32(vv[x][i], p, acc[i]);
    }
  }
  sum = rows4_sum(sum);
  if (!qok) return;
  const float inv = 1.0f / sum;
#pragma unroll
  for (int i = 0; i < NB; ++i) st4(o + pq * E + hd + 16 * i + 4 * lg, acc[i] * inv);
  if (lg == 0) lse[pq * g.heads + F.head] = mx + log2f(sum);
}

// The wave's 16 cells first as queries (dQ, over every key), then as keys (dK, dV, over every
// query).
template <class T, int D>
__global__ __launch_bounds__(256) void k_f32_feat_bwd(Geo g, const T* __restrict__ qkv,
                                                      const T* __restrict__ o,
                                                      const T* __restrict__ dout,
                                                      const float* __restrict__ lse,
                                                      T* __restrict__ dqkv) {
  constexpr int NB = D / 16;
  const FeatTask F = feat_task(g);
  if (!F.ok) return;
  const int lane = threadIdx.x & 63, lg = lane >> 4, c = lane & 15;
  const int E = g.E, E3 = 3 * E, hd = F.head * D;
  auto cell = [&](int x) { return x < F.S ? (F.col0 + x) * g.R + F.r : (int64_t)0; };
  const float tau = 1.0f / sqrtf((float)D);
  const int kc = F.b0 + c;
  const bool own = kc < F.S;
  const int64_t pc = cell(kc);
  // as queries
  {
    Row<D> qf = ld_row<D>(qkv + pc * E3 + hd, own, lg);
    const Row<D> df = ld_row<D>(dout + pc * E + hd, own, lg);
    const Row<D> of = ld_row<D>(o + pc * E + hd, own, lg);
    const float L = own ? lse[pc * g.heads + F.head] : 0.f;
    float Dr = 0.f;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      qf.v[i] = scale4(qf.v[i], tau * LOG2E);
      Dr += dot4(df.v[i], of.v[i]);
    }
    Dr = rows4_sum(Dr);
    f32x4 acc[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) acc[i] = zero4();
    for (int k0 = 0; k0 < F.S; k0 += 16) {
      const bool kok = k0 + c < F.S;
      const T* kp = qkv + cell(k0 + c) * E3 + E + hd;
      const Row<D> kf = ld_row<D>(kp, kok, lg), vf = ld_row<D>(kp + E, kok, lg);
      float kt[4][NB];
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        const int kk = k0 + 4 * lg + x;
        const T* p = qkv + cell(kk) * E3 + E + hd + c;
#pragma unroll
        for (int i = 0; i < NB; ++i) kt[x][i] = kk < F.S ? ld(p + 16 * i) : 0.f;
      }
      const f32x4 s = rows_dot<D>(kf, qf), dp = rows_dot<D>(vf, df);
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        const float ds = k0 + 4 * lg + x < F.S ? exp2_hw(s[x] - L) * (dp[x] - Dr) : 0.f;
#pragma unroll
        for (int i = 0; i < NB; ++i) acc[i] = mfma32(kt[x][i], ds, acc[i]);
      }
    }
    if (own) {
#pragma unroll
      for (int i = 0; i < NB; ++i) st4(dqkv + pc * E3 + hd + 16 * i + 4 * lg, acc[i] * tau);
    }
  }
  // as keys
  const Row<D> kf = ld_row<D>(qkv + pc * E3 + E + hd, own, lg);
  const Row<D> vf = ld_row<D>(qkv + pc * E3 + 2 * E + hd, own, lg);
  f32x4 ak[NB], av[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) ak[i] = av[i] = zero4();
  for (int q0 = 0; q0 < F.S; q0 += 16) {
    const bool qok = q0 + c < F.S;
    const int64_t p = cell(q0 + c);
    Row<D> qf = ld_row<D>(qkv + p * E3 + hd, qok, lg);
    const Row<D> df = ld_row<D>(dout + p * E + hd, qok, lg);
    const Row<D> of = ld_row<D>(o + p * E + hd, qok, lg);
#pragma unroll
    for (int i = 0; i < NB; ++i) qf.v[i] = scale4(qf.v[i], tau * LOG2E);
    float qt[4][NB], dt[4][NB], Lx[4];
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      const int qq = q0 + 4 * lg + x;
      const bool ok = qq < F.S;
      const int64_t px = cell(qq);
      Lx[x] = ok ? lse[px * g.heads + F.head] : 0.f;
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        qt[x][i] = ok ? ld(qkv + px * E3 + hd + c + 16 * i) : 0.f;
        dt[x][i] = ok ? ld(dout + px * E + hd + c + 16 * i) : 0.f;
      }
    }
    float Dr = 0.f;
#pragma unroll
    for (int i = 0; i < NB; ++i) Dr += dot4(df.v[i], of.v[i]);
    Dr = rows4_sum(Dr);  // of query q0 + c
    const f32x4 s = rows_dot<D>(qf, kf), dp = rows_dot<D>(df, vf);
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      const float Dx = __shfl(Dr, 4 * lg + x, 64);
      // a query past the end has zero rows: P = 1 adds zeros
      const float pr = exp2_hw(s[x] - Lx[x]);
      const float ds = pr * (dp[x] - Dx);
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        av[i] = mfma32(dt[x][i], pr, av[i]);
        ak[i] = mfma32(qt[x][i], ds, ak[i]);
      }
    }
  }
  if (!own) return;
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    st4(dqkv + pc * E3 + E + hd + 16 * i + 4 * lg, ak[i] * tau);
    st4(dqkv + pc * E3 + 2 * E + hd + 16 * i + 4 * lg, av[i]);
  }
}

int64_t item_threads(int rows) { return (int64_t)((rows + 63) / 64) * 256; }  // of a problem
unsigned item_grid(const Geo& g, int rows) {
  const int64_t np = ((int64_t)g.NC * g.heads + 7) / 8 * 8;
  return (unsigned)(np * ((rows + 63) / 64));
}
int64_t feat_threads(const Geo& g) { return (int64_t)g.heads * ((g.S + 15) / 16) * 64; }  // a row's
unsigned feat_grid(const Geo& g) {
  return (unsigned)(((int64_t)g.B * g.R * g.heads * ((g.S + 15) / 16) + 3) / 4);
}

}  // namespace

#define BY_D(CALL)                             \
  switch (g.d) {                               \
    case 16: CALL(16); break;                  \
    case 32: CALL(32); break;                  \
    case 64: CALL(64); break;                  \
    default: return hipErrorInvalidValue;      \
  }                                            \
  return hipGetLastError()

template <class T>
hipError_t launch_f32_item_fwd(const Geo& g, const T* q, const T* k, const T* v, T* o, float* lse,
                               hipStream_t s) {
#define CALL(D)                                                                              \
  by_columns(g, item_threads(g.R), [&](const Geo& p, int64_t c0) {                           \
    const int64_t h = c0 * g.heads * g.R;                                                    \
    k_f32_item_fwd<T, D><<<item_grid(p, g.R), 256, 0, s>>>(                                  \
        p, q + h * D, k + h * D, v + h * D, o + c0 * g.R * g.E, lse + h);                    \
  })
  BY_D(CALL);
#undef CALL
}

template <class T>
hipError_t launch_f32_item_bwd(const Geo& g, const T* q, const T* k, const T* v, const T* o,
                               const T* dout, const float* lse, float* Dbuf, T* dq, T* dk, T* dv,
                               hipStream_t s) {
#define CALL(D)                                                                              \
  by_columns(g, item_threads(g.R), [&](const Geo& p, int64_t c0) {                           \
    const int64_t h = c0 * g.heads * g.R, x = c0 * g.R * g.E;                                \
    k_f32_item_dq<T, D><<<item_grid(p, g.R), 256, 0, s>>>(p, q + h * D, k + h * D,           \
                                                          v + h * D, o + x, dout + x,        \
                                                          lse + h, Dbuf + h, dq + h * D);    \
    k_f32_item_dkv<T, D><<<item_grid(p, g.nmax), 256, 0, s>>>(                               \
        p, q + h * D, k + h * D, v + h * D, dout + x, lse + h, Dbuf + h, dk + h * D,         \
        dv + h * D);                                                                         \
  })
  BY_D(CALL);
#undef CALL
}

template <class T>
hipError_t launch_f32_feat_fwd(const Geo& g, const T* qkv, T* o, float* lse, hipStream_t s) {
#define CALL(D)                                                              \
  by_datasets(g, feat_threads(g), [&](const Geo& p) {                        \
    k_f32_feat_fwd<T, D><<<feat_grid(p), 256, 0, s>>>(p, qkv, o, lse);       \
  })
  BY_D(CALL);
#undef CALL
}

template <class T>
hipError_t launch_f32_feat_bwd(const Geo& g, const T* qkv, const T* o, const T* dout,
                               const float* lse, T* dqkv, hipStream_t s) {
#define CALL(D)                                                                          \
  by_datasets(g, feat_threads(g), [&](const Geo& p) {                                    \
    k_f32_feat_bwd<T, D><<<feat_grid(p), 256, 0, s>>>(p, qkv, o, dout, lse, dqkv);       \
  })
  BY_D(CALL);
#undef CALL
}

#define INST(T)                                                                                \
  template hipError_t launch_f32_item_fwd<T>(const Geo&, const T*, const T*, const T*, T*,     \
                                             float*, hipStream_t);                             \
  template hipError_t launch_f32_item_bwd<T>(const Geo&, const T*, const T*, const T*,         \
                                             const T*, const T*, const float*, float*, T*, T*, \
                                             T*, hipStream_t);                                 \
  template hipError_t launch_f32_feat_fwd<T>(const Geo&, const T*, T*, float*, hipStream_t);   \
  template hipError_t launch_f32_feat_bwd<T>(const Geo&, const T*, const T*, const T*,         \
                                             const float*, T*, hipStream_t);
INST(float)
INST(bf16)

}  // namespace tfm
