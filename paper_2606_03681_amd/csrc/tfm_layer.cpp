// Host side of the C ABI declared in include/tfm_layer.h: argument validation, the
// active-cell plan, buffer layouts and the launch sequences of the forward and backward pass.
#include "tfm_layer.h"
#include "tfm_prof.h"

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdarg>
#include <cstdint>
#include <cstdio>
#include <algorithm>
#include <cstring>
#include <numeric>
#include <string>
#include <vector>

#include "kernels.h"
#include "attn.h"
#include "f32.h"
#include "fast.h"
#include "prof.h"
#include "reduce.h"
#include "setup.h"
#include "static_scratch.h"

namespace {

thread_local std::string g_err;

int fail(int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_err = buf;
  return code;
}

constexpr size_t kAlign = 256;
constexpr int64_t kMaxCells = int64_t(1) << 26;

size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

struct Dims {
  int B, R, C, S, E, heads, d, H, dtype;
  int block;       // TFM_BLOCK_POSTNORM or TFM_BLOCK_PRENORM
  float decay;     // pre-norm block: factor on the block input
  size_t tsz;      // bytes per stored element
  int64_t Nmax;    // B * R * S
  int words;       // 32-bit mask words per dataset
};

int check_dims(const tfm_dims* p, Dims& d) {
  if (!p) return fail(TFM_ERR_POINTER, "dims is null");
  d.B = p->B; d.R = p->R; d.C = p->C; d.E = p->E; d.heads = p->heads; d.H = p->H;
  d.dtype = p->dtype;
  if (d.dtype != TFM_F32 && d.dtype != TFM_BF16)
    return fail(TFM_ERR_DIMS, "dtype %d is neither TFM_F32 nor TFM_BF16", d.dtype);
  if (d.B < 1 || d.R < 1) return fail(TFM_ERR_DIMS, "B=%d and R=%d must be >= 1", d.B, d.R);
  if (d.C < 0 || d.C > 255) return fail(TFM_ERR_DIMS, "C=%d outside [0, 255]", d.C);
  if (d.E < 32 || d.E > 256 || d.E % 32)
    return fail(TFM_ERR_DIMS, "E=%d must be a multiple of 32 in [32, 256]", d.E);
  if (d.H < 32 || d.H > 1024 || d.H % 32)
    return fail(TFM_ERR_DIMS, "H=%d must be a multiple of 32 in [32, 1024]", d.H);
  if (d.heads < 1 || d.E % d.heads)
    return fail(TFM_ERR_HEAD_DIM, "E=%d is not a multiple of heads=%d", d.E, d.heads);
  d.d = d.E / d.heads;
  if (d.d != 16 && d.d != 32 && d.d != 64)
    return fail(TFM_ERR_HEAD_DIM, "head dim E/heads=%d not supported (16, 32 or 64)", d.d);
  d.S = d.C + 1;
  d.Nmax = (int64_t)d.B * d.R * d.S;
  if (d.Nmax > kMaxCells)
    return fail(TFM_ERR_DIMS, "B*R*(C+1)=%lld cells exceeds %lld", (long long)d.Nmax,
                (long long)kMaxCells);
  // the attention kernels address one dataset's bf16 Q|K|V [C+1][R][3E] through 32-bit
  // buffer offsets
  if ((int64_t)d.R * d.S * 3 * d.E * 2 > (int64_t)UINT32_MAX)
    return fail(TFM_ERR_DIMS, "R*(C+1)*E=%lld: one dataset's Q|K|V would exceed 4 GiB",
                (long long)d.R * d.S * d.E);
  d.tsz = d.dtype == TFM_F32 ? 4 : 2;
  d.words = (d.S + 31) / 32;
  d.block = p->block;
  d.decay = p->decay;
  if (d.block != TFM_BLOCK_POSTNORM && d.block != TFM_BLOCK_PRENORM)
    return fail(TFM_ERR_DIMS, "block %d is neither TFM_BLOCK_POSTNORM nor TFM_BLOCK_PRENORM",
                d.block);
  if (d.block == TFM_BLOCK_PRENORM) {
    if (d.dtype != TFM_BF16 || !(d.E == 64 || d.E == 128 || d.E == 192 || d.E == 256) ||
        d.H % d.E)
      return fail(TFM_ERR_DIMS, "the pre-norm block needs TFM_BF16, E in {64, 128, 192, 256} "
                                "and H a multiple of E");
    if (!std::isfinite(d.decay)) return fail(TFM_ERR_DIMS, "decay must be finite");
  }
  return TFM_OK;
}

// Dims of the bfloat16 matrix-core path.
bool fast_eligible(const Dims& d) {
  return d.dtype == TFM_BF16 && (d.E == 64 || d.E == 128 || d.E == 192 || d.E == 256) &&
         d.H % d.E == 0;
}

// ---- parameter offsets (floats) -------------------------------------------------------------
struct POff {
  size_t Wqkv_f, bqkv_f, Wo_f, bo_f, Wqkv_i, bqkv_i, Wo_i, bo_i, W1, b1, W2, b2;
  size_t g1, be1, g2, be2, g3, be3, total;
};

// Packed order of include/tfm_layer.h; the pre-norm block has RMSNorm weights g1, g2, g3 only
// (its be* offsets are unused).
POff param_offsets(int E, int H, int block = TFM_BLOCK_POSTNORM) {
  POff o;
  size_t x = 0;
  auto take = [&](size_t n) { size_t r = x; x += n; return r; };
  o.Wqkv_f = take((size_t)3 * E * E); o.bqkv_f = take(3 * E);
  o.Wo_f = take((size_t)E * E); o.bo_f = take(E);
  o.Wqkv_i = take((size_t)3 * E * E); o.bqkv_i = take(3 * E);
  o.Wo_i = take((size_t)E * E); o.bo_i = take(E);
  o.W1 = take((size_t)H * E); o.b1 = take(H);
  o.W2 = take((size_t)E * H); o.b2 = take(E);
  if (block == TFM_BLOCK_PRENORM) {
    o.g1 = take(E); o.g2 = take(E); o.g3 = take(E);
    o.be1 = o.be2 = o.be3 = 0;
  } else {
    o.g1 = take(E); o.be1 = take(E); o.g2 = take(E); o.be2 = take(E);
    o.g3 = take(E); o.be3 = take(E);
  }
  o.total = x;
  return o;
}

// ---- buffer layouts --------------------------------------------------------------------------
struct Arena {
  size_t off = 0;
  size_t take(size_t bytes) { size_t r = off; off = align_up(off + bytes); return r; }
};

// Offsets of the device copy of the plan inside a workspace.
struct MetaOff {
  size_t blob, ds, colmap, col_cell0, col_ntr, cord;
};

MetaOff take_meta(const Dims& d, Arena& a) {
  MetaOff L;
  L.blob = a.take((size_t)d.B * (4 + d.words) * 4);
  L.ds = a.take((size_t)d.B * sizeof(tfm::DsInfo));
  L.colmap = a.take((size_t)d.B * d.S * 4);
  L.col_cell0 = a.take((size_t)d.B * d.S * 8);
  L.col_ntr = a.take((size_t)d.B * d.S * 4);
  L.cord = a.take((size_t)d.B * d.S * 4);
  return L;
}

struct SavedLayout {
  size_t qkvf, of, lsef, h1, xh1, rs1, qi, ki, vi, oi, lsei, h2, xh2, rs2, g, u, xh3, rs3;
  size_t total;
};

SavedLayout saved_layout(const Dims& d) {
  SavedLayout L;
  Arena a;
  const size_t N = (size_t)d.Nmax, t = d.tsz, E = d.E;
  L.qkvf = a.take(N * 3 * E * t);
  L.of = a.take(N * E * t);
  L.lsef = a.take(N * d.heads * 4);
  // the float32-arithmetic path (either storage type) keeps H and x-hat of LN1 and LN2; the MFMA
  // path keeps x-hat only, in the H slots (its LN1 / LN2 affines are folded into the consumers)
  const size_t xhn = fast_eligible(d) ? 0 : N * E * t;
  L.h1 = a.take(N * E * t);
  L.xh1 = a.take(xhn);
  L.rs1 = a.take(N * 4);
  L.qi = a.take(N * E * t);
  L.ki = a.take(N * E * t);
  L.vi = a.take(N * E * t);
  L.oi = a.take(N * E * t);
  L.lsei = a.take(N * d.heads * 4);
  L.h2 = a.take(N * E * t);
  L.xh2 = a.take(xhn);
  L.rs2 = a.take(N * 4);
  // the fused MLP backward recomputes G and U: no saved copies
  const size_t gun = d.dtype == TFM_BF16 && tfm::mlp_fused_ok(d.E, d.H) ? 0 : N * d.H * t;
  L.g = a.take(gun);
  L.u = a.take(gun);
  L.xh3 = a.take(N * E * t);
  L.rs3 = a.take(N * 4);
  L.total = a.off;
  return L;
}

// Saved state of the pre-norm block: x' = decay X, r1 = RMS1(x'), the residual stream h1, h2
// and the norm outputs r2, r3 (the GEMM inputs), rstd of each norm, the attention state and
// the MLP pre-activation and activation.
struct PreSaved {
  size_t xs, r1, rs1, qkvf, of, lsef, h1, r2, rs2, qi, ki, vi, oi, lsei, h2, r3, rs3, g, u;
  size_t total;
};

PreSaved pre_saved_layout(const Dims& d) {
  PreSaved L;
  Arena a;
  const size_t N = (size_t)d.Nmax, t = d.tsz, E = d.E;
  L.xs = a.take(N * E * t);
  L.r1 = a.take(N * E * t);
  L.rs1 = a.take(N * 4);
  L.qkvf = a.take(N * 3 * E * t);
  L.of = a.take(N * E * t);
  L.lsef = a.take(N * d.heads * 4);
  L.h1 = a.take(N * E * t);
  L.r2 = a.take(N * E * t);
  L.rs2 = a.take(N * 4);
  L.qi = a.take(N * E * t);
  L.ki = a.take(N * E * t);
  L.vi = a.take(N * E * t);
  L.oi = a.take(N * E * t);
  L.lsei = a.take(N * d.heads * 4);
  L.h2 = a.take(N * E * t);
  L.r3 = a.take(N * E * t);
  L.rs3 = a.take(N * 4);
  L.g = a.take(N * d.H * t);
  L.u = a.take(N * d.H * t);
  L.total = a.off;
  return L;
}

size_t saved_total(const Dims& d) {
  return d.block == TFM_BLOCK_PRENORM ? pre_saved_layout(d).total : saved_layout(d).total;
}

struct WsLayout {
  MetaOff meta;
  size_t ta;            // float32 mode, forward
  size_t tb;            // post-norm block
  size_t tc, te, tf, th1, tq, tk, tv, tqkv, D;
  size_t th2;           // fused MLP: U for the weight gradient
  size_t part, lnpart;  // float32 mode: weight / bias partials, norm partials
  size_t fast;          // region owned by the MFMA path
  size_t total;
};

WsLayout ws_layout(const Dims& d) {
  WsLayout L;
  Arena a;
  const size_t N = (size_t)d.Nmax, t = d.tsz, E = d.E;
  L.meta = take_meta(d, a);
  const bool f32 = !fast_eligible(d), pre = d.block == TFM_BLOCK_PRENORM;
  L.ta = a.take(f32 ? N * E * t : 0);
  L.tb = a.take(pre ? 0 : N * E * t);
  L.tc = a.take(N * E * t);
  L.te = a.take(N * E * t);
  L.tf = a.take(N * E * t);
  L.th1 = a.take(N * d.H * t);
  L.th2 = a.take(!f32 && !pre && tfm::mlp_fused_ok(d.E, d.H) ? N * d.H * t : 0);
  L.tq = a.take(N * E * t);
  L.tk = a.take(N * E * t);
  L.tv = a.take(N * E * t);
  L.tqkv = a.take(N * 3 * E * t);
  L.D = a.take(N * d.heads * 4);
  L.part = a.take(f32 ? tfm::f32_wpart_floats(d.Nmax, d.E, d.H) * 4 : 0);
  L.lnpart = a.take(f32 ? tfm::f32_lnpart_floats(d.Nmax, d.E) * 4 : 0);
  L.fast = a.take(f32 ? 0 : tfm::fast_workspace_bytes(d.Nmax, d.E, d.H));
  L.total = a.off;
  return L;
}

bool aligned(const void* p) { return p && ((uintptr_t)p % 16) == 0; }

// ---- per-call plan ---------------------------------------------------------------------------
struct Plan {
  int NC = 0;
  int nmax = 0;  // longest train prefix
  // per dataset: n_train, first active column, active columns, first place in the column order
  // of the item-attention backward (below), mask words
  std::vector<int32_t> blob;
  int stride = 0;
  // Column order of the item-attention backward: the columns that run in the one-kernel form first
  // (nF of them, longest prefix nmaxF), then the others; within each group the longer prefixes
  // first, so the largest problems start earliest and the launches end evenly.  natural: one
  // group, in the order of the columns.
  int nF = 0, nmaxF = 0;
  bool natural = true;
};

// nt_max: the largest allowed n_train (R, or the context rows of a query call).
int make_plan(const Dims& d, const int32_t* n_train, const uint8_t* mask, Plan& P,
              int nt_max = -1) {
  if (nt_max < 0) nt_max = d.R;
  if (!n_train || !mask) return fail(TFM_ERR_POINTER, "n_train or cell_mask is null");
  P.stride = 4 + d.words;
  P.blob.assign((size_t)d.B * P.stride, 0);
  int col = 0;
  for (int b = 0; b < d.B; ++b) {
    if (n_train[b] < 1 || n_train[b] > nt_max)
      return fail(TFM_ERR_NTRAIN, "n_train[%d]=%d outside [1, %d]", b, n_train[b], nt_max);
    const uint8_t* m = mask + (size_t)b * d.S;
    if (!m[d.C]) return fail(TFM_ERR_MASK, "target cell (index C=%d) of dataset %d inactive",
                             d.C, b);
    int32_t* e = &P.blob[(size_t)b * P.stride];
    int cnt = 0;
    for (int c = 0; c < d.S; ++c)
      if (m[c]) {
        ++cnt;
        e[4 + (c >> 5)] |= (int32_t)(1u << (c & 31));
      }
    e[0] = n_train[b];
    if (n_train[b] > P.nmax) P.nmax = n_train[b];
    e[1] = e[3] = col;
    e[2] = cnt;
    col += cnt;
  }
  P.NC = col;
  return TFM_OK;
}

// Whether `problems` (column, head) problems of R rows and at most nmax keys that fit the one-kernel
// item-attention backward should take it.
// The one-kernel form runs a problem per CU and pays for whole rounds of 256 and for whole
// thirds of its 768 keys; the two kernels compute each probability twice but spread over rows and
// keys.  Microseconds as measured over d in {16, 32}, 64 to 768 keys (R = 4/3 of them) and 84 to
// 3,936 problems: a 32-row chunk of a round costs 1.7 / 2.1 / 2.57 (d = 16: 1.75, two problems a
// CU / 1.95 / 2.27) for up to 256 / 512 / 768 keys; the two kernels 20 a call, 0.01 a problem and
// 4.9e-7 (3.9e-7) a score of whole 128 x 128 tiles.  One against two, d = 32: 768 keys 83 / 75 us
// at 126 problems, 166 / 135 at 264, 1,314 / 1,604 at 3,936; 512 keys 712 / 719 at 3,936; 384
// keys 521 / 464; 128 keys 21 / 22 at 264.  Both forms are priced as if every
// prefix were the longest, which overstates the two kernels in batches of unequal ones; the rule
// then keeps the one-kernel form where the other is up to 12 % faster.  Forward + backward, one /
// two / this rule: 16 tables of 64 to 760 labelled rows x 21 cells 1,285 / 1,133 / 1,284 us at
// d = 16 (E = 64), 2,845 / 2,684 / 2,844 at d = 32 (E = 192); 40 of 32 to 250 x 11 at d = 32 1,442 /
// 1,392 / 1,381; 3 of 500 to 900 x 11 544 / 512 / 512.
bool item_attn_bwd_fused_pays(int d, int64_t problems, int R, int nmax) {
  const int third = nmax <= 256 ? 0 : (nmax <= 512 ? 1 : 2);
  const double c32[3] = {1.7, 2.1, 2.57}, c16[3] = {1.75, 1.95, 2.27};
  const int64_t slots = d == 16 && third == 0 ? 512 : 256;
  const double one = (double)((problems + slots - 1) / slots) * ((R + 31) / 32) *
                     (d == 16 ? c16 : c32)[third];
  const double tile = (double)((R + 127) / 128 * 128) * ((nmax + 127) / 128 * 128);
  const double two = 20.0 + (double)problems * (0.01 + tile * (d == 16 ? 3.9e-7 : 4.9e-7));
  return one <= 1.05 * two;
}

// Chooses the form of the item-attention backward for each column and orders the columns for it.
void order_columns(const Dims& d, Plan& P) {
  const int fmax = tfm::item_attn_bwd_fused_max_rows(d.d);
  auto rec = [&](int b) { return &P.blob[(size_t)b * P.stride]; };
  for (int b = 0; b < d.B; ++b)
    if (rec(b)[0] <= fmax) {
      P.nF += rec(b)[2];
      P.nmaxF = std::max(P.nmaxF, rec(b)[0]);
    }
  if (!item_attn_bwd_fused_pays(d.d, (int64_t)P.nF * d.heads, d.R, P.nmaxF)) P.nF = P.nmaxF = 0;
  std::vector<int> order(d.B);
  std::iota(order.begin(), order.end(), 0);
  std::stable_sort(order.begin(), order.end(), [&](int x, int y) {
    const bool fx = rec(x)[0] <= P.nmaxF, fy = rec(y)[0] <= P.nmaxF;
    return fx != fy ? fx : rec(x)[0] > rec(y)[0];
  });
  int place = 0;
  for (int b : order) {
    int32_t* e = rec(b);
    e[3] = place;
    place += e[2];
    P.natural = P.natural && e[3] == e[1];
  }
  P.natural = P.natural && (P.nF == 0 || P.nF == P.NC);
}

#define HIPCHK(...)                                                                     \
  do {                                                                                  \
    hipError_t e_ = (__VA_ARGS__);                                                      \
    if (e_ != hipSuccess)                                                               \
      return fail(TFM_ERR_HIP, "%s failed: %s", #__VA_ARGS__, hipGetErrorString(e_));   \
  } while (0)

#define STEP(name, ...)              \
  do {                               \
    tfm::prof_begin(name, s);        \
    HIPCHK(__VA_ARGS__);             \
    tfm::prof_end(s);                \
  } while (0)

// Zeros at the inactive cells of a native output; nothing to launch when every cell is active.
#define ZERO_INACTIVE(g, out)                                                            \
  do {                                                                                   \
    if ((g).NC < (g).B * (g).S)                                                          \
      STEP("zero_inactive/hbm", tfm::launch_zero_inactive(g, out, sizeof(*(out)), s));   \
  } while (0)

#define STEP_ERR(...)                \
  do {                               \
    const int rc_ = (__VA_ARGS__);   \
    if (rc_ != TFM_OK) return rc_;   \
  } while (0)

// Plan and (w not null) weights on the device, in one launch; g describes them.
int setup_geo(const Dims& d, const Plan& P, char* ws, const MetaOff& W, tfm::Geo& g,
              const tfm::SetupWeights* w, hipStream_t s) {
  g.B = d.B; g.R = d.R; g.S = d.S; g.E = d.E; g.heads = d.heads; g.d = d.d; g.H = d.H;
  g.NC = P.NC;
  g.nmax = P.nmax;
  g.N = (int64_t)P.NC * d.R;
  tfm::SetupPlan p{};
  p.B = d.B; p.R = d.R; p.S = d.S; p.words = d.words; p.blob = P.blob.data();
  p.dblob = (int32_t*)(ws + W.blob);
  g.ds = p.ds = (tfm::DsInfo*)(ws + W.ds);
  g.colmap = p.colmap = (int32_t*)(ws + W.colmap);
  g.col_cell0 = p.col_cell0 = (int64_t*)(ws + W.col_cell0);
  g.col_ntr = p.col_ntr = (int32_t*)(ws + W.col_ntr);
  p.cord = (int32_t*)(ws + W.cord);
  STEP("setup/hbm", tfm::launch_setup(p, w, s));
  return TFM_OK;
}

// Item-attention backward on the MFMA path, in the plan's column order: one-kernel columns, then
// the others through the dQ and dK/dV kernels.
int item_attn_bwd(const Dims& d, const tfm::Geo& g, const Plan& P, char* ws, const MetaOff& M,
                  const tfm::bf16* qi, const tfm::bf16* ki, const tfm::bf16* vi,
                  const tfm::bf16* oi, const tfm::bf16* doi, const float* lsei, float* Dq,
                  tfm::bf16* dq, tfm::bf16* dk, tfm::bf16* dv, hipStream_t s) {
  using namespace tfm;
  const int32_t* dcols = P.natural ? nullptr : (const int32_t*)(ws + M.cord);
  const ColList F{dcols, P.nF};
  const ColList T{dcols ? dcols + P.nF : nullptr, P.NC - P.nF};
  if (P.nF > 0)
    STEP("item_attn_bwd/mfma",
         launch_item_attn_bwd_fused(g, F, P.nmaxF, qi, ki, vi, oi, doi, lsei, dq, dk, dv, s));
  if (P.nF < P.NC) {
    STEP("item_attn_dq/mfma", launch_item_attn_dq(g, T, qi, ki, vi, oi, doi, lsei, Dq, dq, s));
    STEP("item_attn_dkdv/mfma",
         launch_item_attn_dkdv(g, T, qi, ki, vi, oi, doi, lsei, Dq, dk, dv, s));
  }
  return TFM_OK;
}

// ---- float32 mode ----------------------------------------------------------------------------
// A linear layer over every active cell: rows of K values, weights W [N][K].
template <class T>
tfm::F32LinArgs<T> f32_linear(const tfm::Geo& g, const T* A, int amode, int K, const float* W,
                              int N, int epi, T* out) {
  tfm::F32LinArgs<T> a{};
  a.M = g.N; a.N = N; a.K = K; a.A = A; a.amode = amode; a.W = W; a.epi = epi; a.out = out;
  a.g = g;
  return a;
}
// Its input gradient: rows of N values (dY) times the weights W [N][K] of the layer, K outputs.
template <class T>
tfm::F32LinArgs<T> f32_linear_dx(const tfm::Geo& g, const T* dY, int N, const float* W, int K,
                                 int epi, T* out) {
  tfm::F32LinArgs<T> a = f32_linear<T>(g, dY, tfm::ROWS_COMPACT, N, W, K, epi, out);
  a.wt = 1;
  return a;
}

template <class T>
int fwd_simple(const Dims& d, const tfm::Geo& g, const T* X, const float* prm, T* Y, char* sv,
               const SavedLayout& S, char* ws, const WsLayout& W, hipStream_t s) {
  using namespace tfm;
  const POff o = param_offsets(d.E, d.H);
  const int E = d.E, H = d.H;
  T* ta = (T*)(ws + W.ta);
  T* u = (T*)(sv + S.u);
  T* qkvf = (T*)(sv + S.qkvf);
  T* of = (T*)(sv + S.of);
  T* h1 = (T*)(sv + S.h1);
  T* h2 = (T*)(sv + S.h2);
  T* oi = (T*)(sv + S.oi);
  T* gp = (T*)(sv + S.g);
  F32LinArgs<T> a = f32_linear<T>(g, X, ROWS_NATIVE, E, prm + o.Wqkv_f, 3 * E, F32_BIAS, qkvf);
  a.bias = prm + o.bqkv_f;
  STEP("feat_qkv/mfma", launch_f32_linear(a, s));
  STEP("feat_attn_fwd/mfma", launch_f32_feat_fwd<T>(g, qkvf, of, (float*)(sv + S.lsef), s));
  a = f32_linear<T>(g, of, ROWS_COMPACT, E, prm + o.Wo_f, E, F32_BIAS, ta);
  a.bias = prm + o.bo_f;
  STEP("feat_out/mfma", launch_f32_linear(a, s));
  STEP("ln1/hbm", launch_f32_add_ln<T>(g, X, ROWS_NATIVE, ta, prm + o.g1, prm + o.be1, h1,
                                       ROWS_COMPACT, (T*)(sv + S.xh1), (float*)(sv + S.rs1), s));
  a = f32_linear<T>(g, h1, ROWS_COMPACT, E, prm + o.Wqkv_i, 3 * E, F32_ITEM_QKV, (T*)(sv + S.qi));
  a.bias = prm + o.bqkv_i; a.out2 = (T*)(sv + S.ki); a.out3 = (T*)(sv + S.vi);
  STEP("item_qkv/mfma", launch_f32_linear(a, s));
  STEP("item_attn_fwd/mfma", launch_f32_item_fwd<T>(g, (T*)(sv + S.qi), (T*)(sv + S.ki), (T*)(sv + S.vi),
                                        oi, (float*)(sv + S.lsei), s));
  a = f32_linear<T>(g, oi, ROWS_COMPACT, E, prm + o.Wo_i, E, F32_BIAS, ta);
  a.bias = prm + o.bo_i;
  STEP("item_out/mfma", launch_f32_linear(a, s));
  STEP("ln2/hbm", launch_f32_add_ln<T>(g, h1, ROWS_COMPACT, ta, prm + o.g2, prm + o.be2, h2,
                                       ROWS_COMPACT, (T*)(sv + S.xh2), (float*)(sv + S.rs2), s));
  a = f32_linear<T>(g, h2, ROWS_COMPACT, E, prm + o.W1, H, F32_GELU, gp);
  a.bias = prm + o.b1; a.out2 = u;
  STEP("mlp_up/mfma", launch_f32_linear(a, s));
  a = f32_linear<T>(g, u, ROWS_COMPACT, H, prm + o.W2, E, F32_BIAS, ta);
  a.bias = prm + o.b2;
  STEP("mlp_down/mfma", launch_f32_linear(a, s));
  STEP("ln3/hbm", launch_f32_add_ln<T>(g, h2, ROWS_COMPACT, ta, prm + o.g3, prm + o.be3, Y,
                                       ROWS_NATIVE, (T*)(sv + S.xh3), (float*)(sv + S.rs3), s));
  ZERO_INACTIVE(g, Y);
  return TFM_OK;
}

// ---- backward --------------------------------------------------------------------------------
#define CHK(...)                 \
  do {                           \
    int c_ = (__VA_ARGS__);      \
    if (c_ != TFM_OK) return c_; \
  } while (0)

template <class T>
int bwd_simple(const Dims& d, const tfm::Geo& g, const T* X, const float* prm, const char* sv,
               const SavedLayout& S, const T* dY, T* dX, float* grads, int accumulate,
               char* ws, const WsLayout& W, hipStream_t s) {
  using namespace tfm;
  const POff o = param_offsets(d.E, d.H);
  const int E = d.E, H = d.H;
  const int64_t N = g.N;
  T* dz3 = (T*)(ws + W.tb);
  T* tmp = (T*)(ws + W.tc);
  T* dz2 = (T*)(ws + W.te);
  T* dz1 = (T*)(ws + W.tf);
  T* du = (T*)(ws + W.th1);
  T* dqkv = (T*)(ws + W.tqkv);
  const T* h1 = (const T*)(sv + S.h1);
  const T* h2 = (const T*)(sv + S.h2);
  const int lnr = f32_ln_rows(N);
  float* lnp[3];
  for (int i = 0; i < 3; ++i) lnp[i] = (float*)(ws + W.lnpart) + (size_t)i * lnr * 2 * E;
  // LN3, from the native dY
  STEP("ln3_bwd/hbm", launch_f32_ln_bwd<T>(g, dY, ROWS_NATIVE, nullptr, (const T*)(sv + S.xh3),
                                           (const float*)(sv + S.rs3), prm + o.g3, dz3, lnp[2],
                                           s));
  // MLP
  F32LinArgs<T> a = f32_linear_dx<T>(g, dz3, E, prm + o.W2, H, F32_GELU_BWD, du);
  a.aux = (const T*)(sv + S.g);
  STEP("mlp_down_dx/mfma", launch_f32_linear(a, s));
  STEP("mlp_up_dx/mfma",
       launch_f32_linear(f32_linear_dx<T>(g, du, H, prm + o.W1, E, F32_BIAS, tmp), s));
  // LN2
  STEP("ln2_bwd/hbm", launch_f32_ln_bwd<T>(g, dz3, ROWS_COMPACT, tmp, (const T*)(sv + S.xh2),
                                           (const float*)(sv + S.rs2), prm + o.g2, dz2, lnp[1],
                                           s));
  // item attention
  T* doi = (T*)(ws + W.tc);
  STEP("item_out_dx/mfma",
       launch_f32_linear(f32_linear_dx<T>(g, dz2, E, prm + o.Wo_i, E, F32_BIAS, doi), s));
  T* dq = (T*)(ws + W.tq);
  T* dk = (T*)(ws + W.tk);
  T* dv = (T*)(ws + W.tv);
  STEP("item_attn_bwd/mfma", launch_f32_item_bwd<T>(g, (const T*)(sv + S.qi), (const T*)(sv + S.ki),
                                        (const T*)(sv + S.vi), (const T*)(sv + S.oi), doi,
                                        (const float*)(sv + S.lsei), (float*)(ws + W.D), dq, dk,
                                        dv, s));
  a = f32_linear_dx<T>(g, dq, 3 * E, prm + o.Wqkv_i, E, F32_BIAS, tmp);
  a.amode = ROWS_ITEM_HM; a.A2 = dk; a.A3 = dv;
  STEP("item_qkv_dx/mfma", launch_f32_linear(a, s));
  // LN1
  STEP("ln1_bwd/hbm", launch_f32_ln_bwd<T>(g, dz2, ROWS_COMPACT, tmp, (const T*)(sv + S.xh1),
                                           (const float*)(sv + S.rs1), prm + o.g1, dz1, lnp[0],
                                           s));
  // feature attention
  T* dof = (T*)(ws + W.tc);
  STEP("feat_out_dx/mfma",
       launch_f32_linear(f32_linear_dx<T>(g, dz1, E, prm + o.Wo_f, E, F32_BIAS, dof), s));
  STEP("feat_attn_bwd/mfma", launch_f32_feat_bwd<T>(g, (const T*)(sv + S.qkvf), (const T*)(sv + S.of), dof,
                                        (const float*)(sv + S.lsef), dqkv, s));
  // every weight and bias gradient in one launch (their operands are all still there; before dX
  // is written, which may share memory with X), and the sums of all partials in another
  const F32Split sp = f32_split(N, E, H);
  F32WgradArgs<T> wa{};
  ReduceList rl;
  wa.g = g;
  float* part = (float*)(ws + W.part);
  auto wgrad = [&](const T* Y, const T* Y2, const T* Y3, int Nj, const T* Xm, int Kj, int xmode,
                   size_t offW, size_t offb) {
    F32WgradJob<T>& j = wa.j[wa.n++];
    j = F32WgradJob<T>{Y, Y2, Y3, Xm, part, part + (size_t)sp.Z * Nj * Kj, Nj, Kj,
                       Y2 ? ROWS_ITEM_HM : ROWS_COMPACT, xmode, 0, 0};
    part = j.bpart + (size_t)sp.Z * Nj;
    rl.add(j.part, (int64_t)Nj * Kj, sp.Z, (int64_t)Nj * Kj, grads + offW);
    rl.add(j.bpart, Nj, sp.Z, Nj, grads + offb);
  };
  wgrad(dqkv, nullptr, nullptr, 3 * E, X, E, ROWS_NATIVE, o.Wqkv_f, o.bqkv_f);
  wgrad(dz1, nullptr, nullptr, E, (const T*)(sv + S.of), E, ROWS_COMPACT, o.Wo_f, o.bo_f);
  wgrad(dq, dk, dv, 3 * E, h1, E, ROWS_COMPACT, o.Wqkv_i, o.bqkv_i);
  wgrad(dz2, nullptr, nullptr, E, (const T*)(sv + S.oi), E, ROWS_COMPACT, o.Wo_i, o.bo_i);
  wgrad(du, nullptr, nullptr, H, h2, E, ROWS_COMPACT, o.W1, o.b1);
  wgrad(dz3, nullptr, nullptr, E, (const T*)(sv + S.u), H, ROWS_COMPACT, o.W2, o.b2);
  // norm scales and shifts are adjacent in the packed order: one sum over 2E columns each
  const size_t og[3] = {o.g1, o.g2, o.g3};
  for (int i = 0; i < 3; ++i) rl.add(lnp[i], 2 * E, lnr, 2 * E, grads + og[i]);
  STEP("wgrad/mfma", launch_f32_wgrads<T>(wa, sp, s));
  a = f32_linear_dx<T>(g, dqkv, 3 * E, prm + o.Wqkv_f, E, F32_DX, dX);
  a.aux = dz1;
  STEP("feat_qkv_dx/mfma", launch_f32_linear(a, s));
  ZERO_INACTIVE(g, dX);
  STEP("reduce/hbm", launch_reduce_list(rl, accumulate, s));
  return TFM_OK;
}

// ---- MFMA path (bfloat16) -------------------------------------------------------------------
struct FastWs {
  tfm::bf16* w;
  tfm::bf16* wt;     // transposed weights (a backward's; null in forward-only calls)
  float* lnpart[3];  // column partials of norm 1, 2, 3 (2 and 3 adjacent)
  float* wpart;      // weight and bias partials
  tfm::WOff wo;
};

FastWs fast_ws(const Dims& d, char* ws, const WsLayout& W) {
  FastWs f;
  f.wo = tfm::weight_offsets(d.E, d.H);
  char* p = ws + W.fast;
  f.w = (tfm::bf16*)p;
  p += align_up((size_t)f.wo.total * 2);
  f.wt = (tfm::bf16*)p;
  p += align_up((size_t)f.wo.total * 2);
  const int64_t ln = tfm::ln_part_floats(d.Nmax, d.E);
  for (int i = 0; i < 3; ++i) f.lnpart[i] = (float*)p + i * ln;
  p += align_up(3 * (size_t)ln * 4);
  f.wpart = (float*)p;
  return f;
}

tfm::GemmArgs gemm_base(const tfm::Geo& g, int64_t M, int N, int K, int epi) {
  tfm::GemmArgs a{};
  a.M = M;
  a.N = N;
  a.K = K;
  a.BN = g.E;
  a.epi = epi;
  a.g = g;
  return a;
}

// Buffers of one forward pass on the MFMA path.  The training forward points them into the
// saved state; the forward-only calls point them into the workspace (reused where lifetimes
// allow; the optional ones null) and into the caller's key/value cache.  h1, h2: in the
// post-norm block the x-hat of LN1 and LN2 (their affines are folded into the consumers); in
// the pre-norm block the residual stream.
struct FwdBufs {
  tfm::bf16 *qkvf = nullptr, *of = nullptr, *h1 = nullptr, *qi = nullptr, *ki = nullptr,
            *vi = nullptr, *oi = nullptr, *h2 = nullptr, *u = nullptr;
  tfm::bf16 *xh3 = nullptr, *g = nullptr;  // optional
  tfm::bf16 *xs = nullptr, *r1 = nullptr, *r2 = nullptr, *r3 = nullptr;    // pre-norm block
  float *lsef = nullptr, *lsei = nullptr, *rs1 = nullptr, *rs2 = nullptr, *rs3 = nullptr;
  bool query = false;  // ki / vi hold the keys and values of a context call: project Q only
  int kR = 0;          // rows per (column, head) of ki / vi; 0: R
  bool save = true;    // the forward keeps what its backward reads (false: forward-only calls)
};

FwdBufs bufs_from_saved(char* sv, const SavedLayout& S) {
  typedef tfm::bf16 T;
  FwdBufs b;
  b.qkvf = (T*)(sv + S.qkvf); b.of = (T*)(sv + S.of); b.lsef = (float*)(sv + S.lsef);
  b.h1 = (T*)(sv + S.h1); b.rs1 = (float*)(sv + S.rs1);
  b.qi = (T*)(sv + S.qi); b.ki = (T*)(sv + S.ki); b.vi = (T*)(sv + S.vi);
  b.oi = (T*)(sv + S.oi); b.lsei = (float*)(sv + S.lsei);
  b.h2 = (T*)(sv + S.h2); b.rs2 = (float*)(sv + S.rs2);
  b.g = (T*)(sv + S.g); b.u = (T*)(sv + S.u); b.xh3 = (T*)(sv + S.xh3);
  b.rs3 = (float*)(sv + S.rs3);
  return b;
}

// Feature Q|K|V (projection of the layer input x, rows per xmode), then the feature attention.
int feat_fwd(const tfm::Geo& g, const tfm::bf16* x, int xmode, const float* bqkv,
             const FwdBufs& b, const FastWs& f, hipStream_t s) {
  using namespace tfm;
  GemmArgs a = gemm_base(g, g.N, 3 * g.E, g.E, EPI_BIAS);
  a.A = x; a.amode = xmode; a.lda = g.E;
  a.Bt = f.w + f.wo.qkv_f; a.bias = bqkv; a.out = b.qkvf; a.ldo = 3 * g.E;
  STEP("feat_qkv/mfma", launch_gemm(a, s));
  if (feat_attn_mfma_ok(g))
    STEP("feat_attn_fwd/mfma", launch_feat_attn_fwd(g, b.qkvf, b.of, b.lsef, s));
  else
    STEP("feat_attn_fwd/mfma", launch_f32_feat_fwd<bf16>(g, b.qkvf, b.of, b.lsef, s));
  return TFM_OK;
}

// What the setup of a forward or backward call on the MFMA path prepares: the matrices it reads
// as stored (forward) or transposed (backward), the LayerNorm folds of the post-norm block, and
// the fused MLP's weight stream in place of the matrices that are in it.  The fused backward
// recomputes G with the folded up-projection bias.
tfm::SetupWeights setup_weights(const Dims& d, const float* prm, const FastWs& f, bool bwd) {
  const POff o = param_offsets(d.E, d.H, d.block);
  tfm::SetupWeights w{};
  w.params = prm; w.E = d.E; w.H = d.H;
  w.wout = f.w; w.wtout = f.wt;
  const bool post = d.block == TFM_BLOCK_POSTNORM;
  const bool fused = post && tfm::mlp_fused_ok(d.E, d.H);
  if (post) w.f = tfm::WFold{prm + o.g1, prm + o.be1, prm + o.bqkv_i, prm + o.g2, prm + o.be2,
                             prm + o.b1};
  if (!bwd) {
    w.w = fused ? 0x07 : 0x3f;  // Wqkv_f, Wo_f, Wqkv_i; Wo_i, W1, W2 unless in the stream
    w.fold = post;
    w.stream = fused ? 1 : 0;
  } else {
    w.wt = fused ? 0x0f : 0x3f;
    w.fold = fused;
    w.stream = fused ? 2 : 0;
  }
  return w;
}

int fwd_fast(const Dims& d, const tfm::Geo& g, const tfm::bf16* X, const float* prm,
             tfm::bf16* Y, const FwdBufs& b, const FastWs& f, hipStream_t s) {
  using namespace tfm;
  const POff o = param_offsets(d.E, d.H);
  const int E = d.E, H = d.H;
  const int64_t N = g.N;
  // H1 and H2 are kept as their x-hat only: the affines of LN1 and LN2 are folded into the
  // products that read them (weights and biases, by the setup) and into the residual reads
  const float* fb = reinterpret_cast<const float*>(f.w + f.wo.fb);
  // feature Q|K|V from the native cells, and the feature attention
  STEP_ERR(feat_fwd(g, X, ROWS_NATIVE, prm + o.bqkv_f, b, f, s));
  // x-hat1 of H1 = LN1(X + O_f Wo_f^T + bo_f)
  GemmArgs a = gemm_base(g, N, E, E, EPI_LN);
  a.A = b.of; a.lda = E; a.Bt = f.w + f.wo.o_f; a.bias = prm + o.bo_f;
  a.resid = X; a.rmode = ROWS_NATIVE; a.gamma = prm + o.g1; a.beta = prm + o.be1;
  a.out = b.h1; a.omode = ROWS_COMPACT; a.xhat_out = 1; a.rstd = b.rs1;
  STEP("feat_out_ln1/mfma", launch_gemm(a, s));
  // item Q (all rows), K, V (train rows), head-major, from x-hat1 with the folded weights;
  // Q only when K/V come from a context call
  a = gemm_base(g, N, b.query ? E : 3 * E, E, EPI_ITEM_QKV);
  a.A = b.h1; a.lda = E; a.Bt = f.w + f.wo.qkv_i; a.bias = fb;
  a.out = b.qi; a.out2 = b.ki; a.out3 = b.vi;
  STEP("item_qkv/mfma", launch_gemm(a, s));
  STEP("item_attn_fwd/mfma",
       launch_item_attn_fwd(g, b.qi, b.ki, b.vi, b.oi, b.lsei, s, b.kR));
  if (mlp_fused_ok(E, H)) {
    // out-projection + LN2, MLP and LN3 in one kernel, the hidden layer in registers
    bf16* ms = f.w + f.wo.ms;
    MlpFwdArgs m{};
    m.M = N; m.oi = b.oi; m.xh1 = b.h1; m.ws = ms;
    m.bo = prm + o.bo_i; m.g1 = prm + o.g1; m.be1 = prm + o.be1; m.g2 = prm + o.g2;
    m.be2 = prm + o.be2; m.b2 = prm + o.b2; m.g3 = prm + o.g3; m.be3 = prm + o.be3;
    m.fb1 = fb + 3 * E;
    // saved for the backward only (G and U are recomputed by the fused backward)
    m.xh2 = b.save ? b.h2 : nullptr; m.rs2 = b.save ? b.rs2 : nullptr;
    m.y = Y; m.xh3 = b.save ? b.xh3 : nullptr; m.rs3 = b.save ? b.rs3 : nullptr; m.g = g;
    STEP("mlp_fused/mfma", launch_mlp_fwd(m, s));
    ZERO_INACTIVE(g, Y);
    return TFM_OK;
  }
  // x-hat2 of H2 = LN2(H1 + O_i Wo_i^T + bo_i), H1 = g1 x-hat1 + be1
  a = gemm_base(g, N, E, E, EPI_LN);
  a.A = b.oi; a.lda = E; a.Bt = f.w + f.wo.o_i; a.bias = prm + o.bo_i;
  a.resid = b.h1; a.rmode = ROWS_COMPACT; a.rgamma = prm + o.g1; a.rbeta = prm + o.be1;
  a.gamma = prm + o.g2; a.beta = prm + o.be2;
  a.out = b.h2; a.omode = ROWS_COMPACT; a.xhat_out = 1; a.rstd = b.rs2;
  STEP("item_out_ln2/mfma", launch_gemm(a, s));
  // G = H2 W1^T + b1 (from x-hat2, folded), U = GELU(G)
  a = gemm_base(g, N, H, E, EPI_GELU_FWD);
  a.A = b.h2; a.lda = E; a.Bt = f.w + f.wo.w1; a.bias = fb + 3 * E;
  a.out = b.g; a.out2 = b.u; a.ldo = H;
  STEP("mlp_up/mfma", launch_gemm(a, s));
  // Y = LN3(H2 + U W2^T + b2), written to the native layout
  a = gemm_base(g, N, E, H, EPI_LN);
  a.A = b.u; a.lda = H; a.Bt = f.w + f.wo.w2; a.bias = prm + o.b2;
  a.resid = b.h2; a.rmode = ROWS_COMPACT; a.rgamma = prm + o.g2; a.rbeta = prm + o.be2;
  a.gamma = prm + o.g3; a.beta = prm + o.be3;
  a.out = Y; a.omode = ROWS_NATIVE; a.xhat = b.xh3; a.rstd = b.rs3;
  STEP("mlp_down_ln3/mfma", launch_gemm(a, s));
  ZERO_INACTIVE(g, Y);
  return TFM_OK;
}

// Weight, bias and norm gradients of one backward pass on the MFMA path: the passes note them
// as their operands become final (every operand keeps its buffer until then), products() forms
// all products in one launch and sums() adds all partials in another.
struct FastGrads {
  float* wpart;
  float* grads;
  tfm::WgradSplit sp;
  tfm::WgradArgs wa{};
  tfm::ReduceList rl;

  FastGrads(const Dims& d, const tfm::Geo& g, const FastWs& f, float* grads)
      : wpart(f.wpart), grads(grads), sp(tfm::wgrad_split(g.N, d.E, d.H)) {
    wa.g = g;
  }
  // One linear: rows dY (N values; head-major item gradients when dY2 is given) and X (K values).
  // xg, xb: X is the x-hat of a norm with affine (xg, xb), the gradient is formed for
  // xg o X + xb.
  void linear(const tfm::bf16* dY, int N, const tfm::bf16* X, int K, int xmode, size_t offW,
              size_t offb, const tfm::bf16* dY2 = nullptr, const tfm::bf16* dY3 = nullptr,
              int ymode = tfm::ROWS_COMPACT, const float* xg = nullptr,
              const float* xb = nullptr) {
    tfm::WgradJob& j = wa.j[wa.n++];
    j = tfm::WgradJob{N, K, dY, dY2, dY3, X, dY2 ? tfm::ROWS_ITEM_HM : ymode, xmode,
                      wpart, wpart + (size_t)sp.Z * N * K, 0};
    wpart = j.bpart + (size_t)sp.Z * N;
    if (xg)
      rl.add_fold(j.part, (int64_t)N * K, sp.Z, N, K, grads + offW, j.bpart, N, xg, xb);
    else
      rl.add(j.part, (int64_t)N * K, sp.Z, (int64_t)N * K, grads + offW);
    rl.add(j.bpart, N, sp.Z, N, grads + offb);
  }
  // Norm parameters: count column sums from rows of `stride` partials.
  void norm(const float* part, int64_t stride, int rows, int64_t count, size_t off) {
    rl.add(part, stride, rows, count, grads + off);
  }
  // Every product; called before dX is written, which may share memory with X or dY.
  int products(hipStream_t s) {
    STEP("wgrad/mfma", tfm::launch_wgrads(wa, sp, s));
    return TFM_OK;
  }
  int sums(int accumulate, hipStream_t s) {
    STEP("reduce/hbm", tfm::launch_reduce_list(rl, accumulate, s));
    return TFM_OK;
  }
};

int bwd_fast(const Dims& d, const tfm::Geo& g, const Plan& P, const tfm::bf16* X,
             const float* prm, const char* sv, const SavedLayout& S, const tfm::bf16* dY,
             tfm::bf16* dX, float* grads, int accumulate, char* ws, const WsLayout& W,
             hipStream_t s) {
  using namespace tfm;
  typedef tfm::bf16 T;
  const POff o = param_offsets(d.E, d.H);
  const FastWs f = fast_ws(d, ws, W);
  const int E = d.E, H = d.H;
  const int64_t N = g.N;
  const int tiles = (int)tfm::gemm_tiles(tfm::EPI_LN_BWD, E, N);
  FastGrads G(d, g, f, grads);
  const bool fused_mlp = mlp_fused_ok(E, H);
  T* dz3 = (T*)(ws + W.tb);
  T* dz2 = (T*)(ws + W.te);
  T* dz1 = (T*)(ws + W.tf);
  T* dgb = (T*)(ws + W.th1);
  T* dqkv = (T*)(ws + W.tqkv);
  const T* xh1 = (const T*)(sv + S.h1);  // the forward keeps x-hat1 and x-hat2 only
  const T* xh2 = (const T*)(sv + S.h2);
  if (fused_mlp) {
    // LN3', the MLP backward with G recomputed, LN2' in one kernel; its column sums give the
    // LN3 and LN2 weight and bias gradients (each pair adjacent in the packed order)
    T* ub = (T*)(ws + W.th2);
    bf16* ms = f.w + f.wo.ms;
    MlpBwdArgs m{};
    m.M = N; m.dy = dY; m.xh3 = (const T*)(sv + S.xh3); m.rs3 = (const float*)(sv + S.rs3);
    m.xh2 = xh2; m.rs2 = (const float*)(sv + S.rs2); m.ws = ms;
    m.g3 = prm + o.g3; m.g2 = prm + o.g2;
    m.fb1 = reinterpret_cast<const float*>(f.w + f.wo.fb) + 3 * E;
    m.dz3 = dz3; m.dz2 = dz2; m.dg = dgb; m.u = ub; m.part = f.lnpart[1]; m.g = g;
    STEP("mlp_bwd_fused/mfma", launch_mlp_bwd(m, s));
    const int nt = (int)mlp_bwd_tiles(N);
    G.norm(f.lnpart[1], 4 * E, nt, 2 * E, o.g3);
    G.norm(f.lnpart[1] + 2 * E, 4 * E, nt, 2 * E, o.g2);
    G.linear(dz3, E, ub, H, ROWS_COMPACT, o.W2, o.b2);
    G.linear(dgb, H, xh2, E, ROWS_COMPACT, o.W1, o.b1, nullptr, nullptr, ROWS_COMPACT,
              prm + o.g2, prm + o.be2);
  } else {
    // LN3 (from the native dY), with its gamma/beta column sums
    int nb = 0;
    STEP("ln3_bwd/hbm", launch_ln_out_bwd(g, dY, (const T*)(sv + S.xh3),
                                          (const float*)(sv + S.rs3), prm + o.g3, dz3, f.lnpart[2],
                                          &nb, s));
    // gamma and beta gradients are adjacent in the packed order: one sum over 2E columns
    G.norm(f.lnpart[2], 2 * E, nb, 2 * E, o.g3);
    // MLP: dG = (dZ3 W2) * GELU'(G)
    GemmArgs a = gemm_base(g, N, H, E, EPI_GELU_BWD);
    a.A = dz3; a.lda = E; a.Bt = f.wt + f.wo.w2; a.out = dgb; a.ldo = H;
    a.aux = (const T*)(sv + S.g);
    STEP("mlp_down_dx/mfma", launch_gemm(a, s));
    G.linear(dz3, E, (const T*)(sv + S.u), H, ROWS_COMPACT, o.W2, o.b2);
    G.linear(dgb, H, xh2, E, ROWS_COMPACT, o.W1, o.b1, nullptr, nullptr, ROWS_COMPACT,
              prm + o.g2, prm + o.be2);
    // dZ2 = LN2'(dZ3 + dG W1)
    a = gemm_base(g, N, E, H, EPI_LN_BWD);
    a.A = dgb; a.lda = H; a.Bt = f.wt + f.wo.w1; a.resid = dz3; a.aux = xh2;
    a.rstd_in = (const float*)(sv + S.rs2); a.gamma = prm + o.g2; a.out = dz2; a.part = f.lnpart[1];
    STEP("mlp_up_dx_ln2/mfma", launch_gemm(a, s));
    G.norm(f.lnpart[1], 2 * E, tiles, 2 * E, o.g2);
  }
  GemmArgs a;
  // item attention
  T* doi = (T*)(ws + W.tc);
  a = gemm_base(g, N, E, E, EPI_BIAS);
  a.A = dz2; a.lda = E; a.Bt = f.wt + f.wo.o_i; a.out = doi; a.ldo = E;
  STEP("item_out_dx/mfma", launch_gemm(a, s));
  G.linear(dz2, E, (const T*)(sv + S.oi), E, ROWS_COMPACT, o.Wo_i, o.bo_i);
  T* dq = (T*)(ws + W.tq);
  T* dk = (T*)(ws + W.tk);
  T* dv = (T*)(ws + W.tv);
  const T* qi = (const T*)(sv + S.qi);
  const T* ki = (const T*)(sv + S.ki);
  const T* vi = (const T*)(sv + S.vi);
  const T* oi = (const T*)(sv + S.oi);
  const float* lsei = (const float*)(sv + S.lsei);
  float* Dq = (float*)(ws + W.D);
  CHK(item_attn_bwd(d, g, P, ws, W.meta, qi, ki, vi, oi, doi, lsei, Dq, dq, dk, dv, s));
  G.linear(dq, 3 * E, xh1, E, ROWS_COMPACT, o.Wqkv_i, o.bqkv_i, dk, dv, ROWS_COMPACT,
            prm + o.g1, prm + o.be1);
  // dZ1 = LN1'(dZ2 + dQKV_i Wqkv_i), the gradients read head-major in place
  a = gemm_base(g, N, E, 3 * E, EPI_LN_BWD);
  a.A = dq; a.A2 = dk; a.A3 = dv; a.amode = ROWS_ITEM_HM; a.lda = 3 * E;
  a.Bt = f.wt + f.wo.qkv_i; a.resid = dz2;
  a.aux = xh1; a.rstd_in = (const float*)(sv + S.rs1); a.gamma = prm + o.g1;
  a.out = dz1; a.part = f.lnpart[0];
  STEP("item_qkv_dx_ln1/mfma", launch_gemm(a, s));
  G.norm(f.lnpart[0], 2 * E, tiles, 2 * E, o.g1);
  // feature attention
  T* dof = (T*)(ws + W.tc);
  a = gemm_base(g, N, E, E, EPI_BIAS);
  a.A = dz1; a.lda = E; a.Bt = f.wt + f.wo.o_f; a.out = dof; a.ldo = E;
  STEP("feat_out_dx/mfma", launch_gemm(a, s));
  G.linear(dz1, E, (const T*)(sv + S.of), E, ROWS_COMPACT, o.Wo_f, o.bo_f);
  if (feat_attn_mfma_ok(g))
    STEP("feat_attn_bwd/mfma",
         launch_feat_attn_bwd(g, (const T*)(sv + S.qkvf), (const T*)(sv + S.of), dof,
                              (const float*)(sv + S.lsef), dqkv, s));
  else
    STEP("feat_attn_bwd/mfma", launch_f32_feat_bwd<T>(g, (const T*)(sv + S.qkvf), (const T*)(sv + S.of), dof,
                                        (const float*)(sv + S.lsef), dqkv, s));
  G.linear(dqkv, 3 * E, X, E, ROWS_NATIVE, o.Wqkv_f, o.bqkv_f);
  CHK(G.products(s));
  // dX = dZ1 + dQKV_f Wqkv_f, native layout
  a = gemm_base(g, N, E, 3 * E, EPI_DX);
  a.A = dqkv; a.lda = 3 * E; a.Bt = f.wt + f.wo.qkv_f; a.resid = dz1; a.out = dX;
  STEP("feat_qkv_dx/mfma", launch_gemm(a, s));
  ZERO_INACTIVE(g, dX);
  return G.sums(accumulate, s);
}

// ---- pre-norm RMSNorm block (bfloat16, MFMA path) --------------------------------------------
constexpr float kRmsEps = 1e-6f;

FwdBufs bufs_from_pre_saved(char* sv, const PreSaved& S) {
  typedef tfm::bf16 T;
  FwdBufs b;
  b.xs = (T*)(sv + S.xs); b.r1 = (T*)(sv + S.r1); b.rs1 = (float*)(sv + S.rs1);
  b.qkvf = (T*)(sv + S.qkvf); b.of = (T*)(sv + S.of); b.lsef = (float*)(sv + S.lsef);
  b.h1 = (T*)(sv + S.h1); b.r2 = (T*)(sv + S.r2); b.rs2 = (float*)(sv + S.rs2);
  b.qi = (T*)(sv + S.qi); b.ki = (T*)(sv + S.ki); b.vi = (T*)(sv + S.vi);
  b.oi = (T*)(sv + S.oi); b.lsei = (float*)(sv + S.lsei);
  b.h2 = (T*)(sv + S.h2); b.r3 = (T*)(sv + S.r3); b.rs3 = (float*)(sv + S.rs3);
  b.g = (T*)(sv + S.g); b.u = (T*)(sv + S.u);
  return b;
}

int fwd_pre(const Dims& d, const tfm::Geo& g, const tfm::bf16* X, const float* prm,
            tfm::bf16* Y, const FwdBufs& b, const FastWs& f, hipStream_t s) {
  using namespace tfm;
  const POff o = param_offsets(d.E, d.H, d.block);
  const int E = d.E, H = d.H;
  const int64_t N = g.N;
  // x' = decay X, r1 = RMS1(x')
  STEP("rms_in/hbm", launch_rms_in(g, X, d.decay, prm + o.g1, kRmsEps, b.xs, b.r1, b.rs1, s));
  STEP_ERR(feat_fwd(g, b.r1, ROWS_COMPACT, prm + o.bqkv_f, b, f, s));
  // h1 = x' + O_f Wo_f^T + bo_f, r2 = RMS2(h1)
  GemmArgs a = gemm_base(g, N, E, E, EPI_RMS);
  a.A = b.of; a.lda = E; a.Bt = f.w + f.wo.o_f; a.bias = prm + o.bo_f;
  a.resid = b.xs; a.rmode = ROWS_COMPACT; a.rscale = 1.0f; a.gamma = prm + o.g2;
  a.eps = kRmsEps; a.out = b.h1; a.out2 = b.r2; a.rstd = b.rs2;
  STEP("feat_out_rms2/mfma", launch_gemm(a, s));
  // item Q (all rows), K and V (train rows), head-major; Q only when K/V come from a context
  // call
  a = gemm_base(g, N, b.query ? E : 3 * E, E, EPI_ITEM_QKV);
  a.A = b.r2; a.lda = E; a.Bt = f.w + f.wo.qkv_i; a.bias = prm + o.bqkv_i;
  a.out = b.qi; a.out2 = b.ki; a.out3 = b.vi;
  STEP("item_qkv/mfma", launch_gemm(a, s));
  STEP("item_attn_fwd/mfma",
       launch_item_attn_fwd(g, b.qi, b.ki, b.vi, b.oi, b.lsei, s, b.kR));
  // h2 = h1 + O_i Wo_i^T + bo_i, r3 = RMS3(h2)
  a = gemm_base(g, N, E, E, EPI_RMS);
  a.A = b.oi; a.lda = E; a.Bt = f.w + f.wo.o_i; a.bias = prm + o.bo_i;
  a.resid = b.h1; a.rmode = ROWS_COMPACT; a.rscale = 1.0f; a.gamma = prm + o.g3;
  a.eps = kRmsEps; a.out = b.h2; a.out2 = b.r3; a.rstd = b.rs3;
  STEP("item_out_rms3/mfma", launch_gemm(a, s));
  // G = r3 W1^T + b1, U = GELU(G)
  a = gemm_base(g, N, H, E, EPI_GELU_FWD);
  a.A = b.r3; a.lda = E; a.Bt = f.w + f.wo.w1; a.bias = prm + o.b1;
  a.out = b.g; a.out2 = b.u; a.ldo = H;
  STEP("mlp_up/mfma", launch_gemm(a, s));
  // Y = h2 + U W2^T + b2, native
  a = gemm_base(g, N, E, H, EPI_DX);
  a.A = b.u; a.lda = H; a.Bt = f.w + f.wo.w2; a.bias = prm + o.b2; a.resid = b.h2;
  a.out = Y;
  STEP("mlp_down_res/mfma", launch_gemm(a, s));
  ZERO_INACTIVE(g, Y);
  return TFM_OK;
}

int bwd_pre(const Dims& d, const tfm::Geo& g, const Plan& P, const float* prm, const char* sv,
            const PreSaved& S, const tfm::bf16* dY, tfm::bf16* dX, float* grads, int accumulate,
            char* ws, const WsLayout& W, hipStream_t s) {
  using namespace tfm;
  typedef tfm::bf16 T;
  const POff o = param_offsets(d.E, d.H, d.block);
  const FastWs f = fast_ws(d, ws, W);
  const int E = d.E, H = d.H;
  const int64_t N = g.N;
  const int tiles = (int)tfm::gemm_tiles(tfm::EPI_RMS_BWD, E, N);
  FastGrads G(d, g, f, grads);
  T* dh2 = (T*)(ws + W.te);
  T* dh1 = (T*)(ws + W.tf);
  T* dgb = (T*)(ws + W.th1);
  T* dqkv = (T*)(ws + W.tqkv);
  // dY is read in its native layout by the three steps that need it (no compact copy)
  // dG = (dY W2) * GELU'(G)
  GemmArgs a = gemm_base(g, N, H, E, EPI_GELU_BWD);
  a.A = dY; a.amode = ROWS_NATIVE; a.lda = E; a.Bt = f.wt + f.wo.w2; a.out = dgb; a.ldo = H;
  a.aux = (const T*)(sv + S.g);
  STEP("mlp_down_dx/mfma", launch_gemm(a, s));
  G.linear(dY, E, (const T*)(sv + S.u), H, ROWS_COMPACT, o.W2, o.b2, nullptr, nullptr,
            ROWS_NATIVE);
  G.linear(dgb, H, (const T*)(sv + S.r3), E, ROWS_COMPACT, o.W1, o.b1);
  // dh2 = dY + RMS3'(dG W1)
  a = gemm_base(g, N, E, H, EPI_RMS_BWD);
  a.A = dgb; a.lda = H; a.Bt = f.wt + f.wo.w1; a.resid = dY; a.rmode = ROWS_NATIVE;
  a.aux = (const T*)(sv + S.h2);
  a.rstd_in = (const float*)(sv + S.rs3); a.gamma = prm + o.g3; a.eps = kRmsEps;
  a.oscale = 1.0f; a.omode = ROWS_COMPACT; a.out = dh2; a.part = f.lnpart[2];
  STEP("mlp_up_dx_rms3/mfma", launch_gemm(a, s));
  G.norm(f.lnpart[2], E, tiles, E, o.g3);
  // item attention
  T* doi = (T*)(ws + W.tc);
  a = gemm_base(g, N, E, E, EPI_BIAS);
  a.A = dh2; a.lda = E; a.Bt = f.wt + f.wo.o_i; a.out = doi; a.ldo = E;
  STEP("item_out_dx/mfma", launch_gemm(a, s));
  G.linear(dh2, E, (const T*)(sv + S.oi), E, ROWS_COMPACT, o.Wo_i, o.bo_i);
  T* dq = (T*)(ws + W.tq);
  T* dk = (T*)(ws + W.tk);
  T* dv = (T*)(ws + W.tv);
  const T* qi = (const T*)(sv + S.qi);
  const T* ki = (const T*)(sv + S.ki);
  const T* vi = (const T*)(sv + S.vi);
  const T* oi = (const T*)(sv + S.oi);
  const float* lsei = (const float*)(sv + S.lsei);
  float* Dq = (float*)(ws + W.D);
  CHK(item_attn_bwd(d, g, P, ws, W.meta, qi, ki, vi, oi, doi, lsei, Dq, dq, dk, dv, s));
  G.linear(dq, 3 * E, (const T*)(sv + S.r2), E, ROWS_COMPACT, o.Wqkv_i, o.bqkv_i, dk, dv);
  // dh1 = dh2 + RMS2'(dQKV_i Wqkv_i), the gradients read head-major in place
  a = gemm_base(g, N, E, 3 * E, EPI_RMS_BWD);
  a.A = dq; a.A2 = dk; a.A3 = dv; a.amode = ROWS_ITEM_HM; a.lda = 3 * E;
  a.Bt = f.wt + f.wo.qkv_i; a.resid = dh2; a.aux = (const T*)(sv + S.h1);
  a.rstd_in = (const float*)(sv + S.rs2); a.gamma = prm + o.g2; a.eps = kRmsEps;
  a.oscale = 1.0f; a.omode = ROWS_COMPACT; a.out = dh1; a.part = f.lnpart[1];
  STEP("item_qkv_dx_rms2/mfma", launch_gemm(a, s));
  G.norm(f.lnpart[1], E, tiles, E, o.g2);
  // feature attention
  T* dof = (T*)(ws + W.tc);
  a = gemm_base(g, N, E, E, EPI_BIAS);
  a.A = dh1; a.lda = E; a.Bt = f.wt + f.wo.o_f; a.out = dof; a.ldo = E;
  STEP("feat_out_dx/mfma", launch_gemm(a, s));
  G.linear(dh1, E, (const T*)(sv + S.of), E, ROWS_COMPACT, o.Wo_f, o.bo_f);
  if (feat_attn_mfma_ok(g))
    STEP("feat_attn_bwd/mfma",
         launch_feat_attn_bwd(g, (const T*)(sv + S.qkvf), (const T*)(sv + S.of), dof,
                              (const float*)(sv + S.lsef), dqkv, s));
  else
    STEP("feat_attn_bwd/mfma", launch_f32_feat_bwd<T>(g, (const T*)(sv + S.qkvf), (const T*)(sv + S.of), dof,
                                        (const float*)(sv + S.lsef), dqkv, s));
  G.linear(dqkv, 3 * E, (const T*)(sv + S.r1), E, ROWS_COMPACT, o.Wqkv_f, o.bqkv_f);
  CHK(G.products(s));
  // dX = decay (dh1 + RMS1'(dQKV_f Wqkv_f)), native
  a = gemm_base(g, N, E, 3 * E, EPI_RMS_BWD);
  a.A = dqkv; a.lda = 3 * E; a.Bt = f.wt + f.wo.qkv_f; a.resid = dh1;
  a.aux = (const T*)(sv + S.xs); a.rstd_in = (const float*)(sv + S.rs1); a.gamma = prm + o.g1;
  a.eps = kRmsEps; a.oscale = d.decay; a.omode = ROWS_NATIVE; a.out = dX; a.part = f.lnpart[0];
  STEP("feat_qkv_dx_rms1/mfma", launch_gemm(a, s));
  G.norm(f.lnpart[0], E, tiles, E, o.g1);
  ZERO_INACTIVE(g, dX);
  return G.sums(accumulate, s);
}

// ---- forward-only calls ----------------------------------------------------------------------
// Workspace of a forward-only call: the plan, the bf16 weights, and the activations of one
// pass with lifetimes overlapped (p1: feature Q|K|V, then GELU output; p2: feature attention
// output, then item attention output; p3: h1; p4: item Q, then h2 (post-norm); pre-norm adds
// p5: x', then h2, and p6: r1, then r2, then r3), one rstd and one log-sum-exp scratch.
struct InferLayout {
  MetaOff meta;
  size_t w, p1, p2, p3, p4, p5, p6, rs, lse, total;
};

bool infer_eligible(const Dims& d) {
  return d.dtype == TFM_BF16 && (d.E == 64 || d.E == 128 || d.E == 192 || d.E == 256) &&
         d.H % d.E == 0;
}

InferLayout infer_layout(const Dims& d) {
  InferLayout L;
  Arena a;
  const size_t N = (size_t)d.Nmax, E = d.E;
  const tfm::WOff wo = tfm::weight_offsets(d.E, d.H);
  L.meta = take_meta(d, a);
  L.w = a.take((size_t)wo.total * 2);
  // activations from a 64 KiB boundary on: 16 tables of 768 + 256 rows x 101 cells at E = 192 take
  // 4,880 us so (4,875 from 2 MiB), and 4,910 to 4,935 from other places
  a.off = (a.off + 65535) / 65536 * 65536;
  L.p1 = a.take(N * (3 * E > (size_t)d.H ? 3 * E : (size_t)d.H) * 2);
  L.p2 = a.take(N * E * 2);
  L.p3 = a.take(N * E * 2);
  L.p4 = a.take(N * E * 2);
  const bool pre = d.block == TFM_BLOCK_PRENORM;
  L.p5 = pre ? a.take(N * E * 2) : 0;
  L.p6 = pre ? a.take(N * E * 2) : 0;
  L.rs = a.take(N * 4);
  L.lse = a.take(N * d.heads * 4);
  L.total = a.off;
  return L;
}

// Key/value cache of one layer: K then V, head-major [column][head][R][d] over every possible
// active column (B * (C + 1)), R = the context rows.
size_t cache_half(const Dims& d) { return align_up((size_t)d.B * d.S * d.R * d.E * 2); }

FwdBufs infer_bufs(const Dims& d, char* ws, const InferLayout& L, tfm::bf16* kc, tfm::bf16* vc,
                   bool query, int kR) {
  typedef tfm::bf16 T;
  FwdBufs b;
  T* p1 = (T*)(ws + L.p1);
  T* p2 = (T*)(ws + L.p2);
  T* p3 = (T*)(ws + L.p3);
  T* p4 = (T*)(ws + L.p4);
  float* rs = (float*)(ws + L.rs);
  float* lse = (float*)(ws + L.lse);
  b.qkvf = p1; b.u = p1;
  b.of = p2; b.oi = p2;
  b.h1 = p3;
  b.qi = p4;
  b.ki = kc; b.vi = vc;
  b.lsef = lse; b.lsei = lse;
  b.rs1 = b.rs2 = b.rs3 = rs;
  if (d.block == TFM_BLOCK_PRENORM) {
    T* p5 = (T*)(ws + L.p5);
    T* p6 = (T*)(ws + L.p6);
    b.xs = p5; b.h2 = p5;
    b.r1 = b.r2 = b.r3 = p6;
  } else {
    b.h2 = p4;
  }
  b.query = query;
  b.kR = kR;
  b.save = false;
  return b;
}

FastWs infer_fast_ws(const Dims& d, char* ws, const InferLayout& L) {
  FastWs f{};
  f.wo = tfm::weight_offsets(d.E, d.H);
  f.w = (tfm::bf16*)(ws + L.w);
  return f;
}

// Shared part of the two forward-only calls.  ctx_rows < 0: a context call (dims->R rows, the
// cache written); otherwise a query call whose cache came from a context call with ctx_rows
// rows.
int infer_call(const tfm_dims* dims, int ctx_rows, const int32_t* n_train,
               const uint8_t* cell_mask, const void* X, const float* params, void* Y,
               void* cache, size_t cache_bytes, void* workspace, size_t workspace_bytes,
               hipStream_t s) {
  Dims d;
  int rc = check_dims(dims, d);
  if (rc) return rc;
  if (!infer_eligible(d))
    return fail(TFM_ERR_DIMS, "forward-only calls need TFM_BF16, E in {64, 128, 192, 256} and H "
                              "a multiple of E");
  const bool query = ctx_rows >= 0;
  Dims dc = d;  // the dims the cache was laid out for
  if (query) {
    if (ctx_rows < 1) return fail(TFM_ERR_DIMS, "context_rows=%d must be >= 1", ctx_rows);
    tfm_dims pc = *dims;
    pc.R = ctx_rows;
    rc = check_dims(&pc, dc);
    if (rc) return rc;
  }
  if (!aligned(X) || !aligned(params) || !aligned(Y) || !aligned(cache) || !aligned(workspace))
    return fail(TFM_ERR_POINTER, "X, params, Y, kv_cache and workspace must be non-null and "
                                 "16-byte aligned");
  const InferLayout L = infer_layout(d);
  if (workspace_bytes < L.total)
    return fail(TFM_ERR_BUFFER, "workspace has %zu bytes, %zu required", workspace_bytes,
                L.total);
  if (cache_bytes < 2 * cache_half(dc))
    return fail(TFM_ERR_BUFFER, "kv_cache has %zu bytes, %zu required", cache_bytes,
                2 * cache_half(dc));
  Plan P;
  rc = make_plan(d, n_train, cell_mask, P, query ? ctx_rows : d.R);
  if (rc) return rc;
  char* ws = (char*)workspace;
  tfm::Geo g;
  const FastWs f = infer_fast_ws(d, ws, L);
  const tfm::SetupWeights sw = setup_weights(d, params, f, false);
  rc = setup_geo(d, P, ws, L.meta, g, &sw, s);
  if (rc) return rc;
  tfm::bf16* kc = (tfm::bf16*)cache;
  tfm::bf16* vc = (tfm::bf16*)((char*)cache + cache_half(dc));
  const FwdBufs b = infer_bufs(d, ws, L, kc, vc, query, query ? ctx_rows : d.R);
  if (d.block == TFM_BLOCK_PRENORM)
    return fwd_pre(d, g, (const tfm::bf16*)X, params, (tfm::bf16*)Y, b, f, s);
  return fwd_fast(d, g, (const tfm::bf16*)X, params, (tfm::bf16*)Y, b, f, s);
}

}  // namespace

// ============================================================================ C ABI
namespace tfm {
int abi_fail(int code, const char* msg) { return fail(code, "%s", msg); }
int abi_check_dims(const void* dims) {
  Dims d;
  return check_dims((const tfm_dims*)dims, d);
}
}  // namespace tfm

extern "C" {

size_t tfm_layer_param_count(const tfm_dims* dims) {
  Dims d;
  if (check_dims(dims, d) != TFM_OK) return 0;
  return param_offsets(d.E, d.H, d.block).total;
}

size_t tfm_layer_saved_bytes(const tfm_dims* dims) {
  Dims d;
  if (check_dims(dims, d) != TFM_OK) return 0;
  return saved_total(d);
}

size_t tfm_layer_workspace_bytes(const tfm_dims* dims) {
  Dims d;
  if (check_dims(dims, d) != TFM_OK) return 0;
  return ws_layout(d).total;
}

const char* tfm_last_error(void) { return g_err.c_str(); }

int tfm_prof_item_bwd_fused_rows(int head_dim) {
  return tfm::item_attn_bwd_fused_max_rows(head_dim);
}

int tfm_prof_item_bwd_columns(const tfm_dims* dims, const int32_t* n_train,
                              const uint8_t* cell_mask, int32_t* order) {
  Dims d;
  int rc = check_dims(dims, d);
  if (rc) return rc;
  Plan P;
  rc = make_plan(d, n_train, cell_mask, P);
  if (rc) return rc;
  if (fast_eligible(d)) order_columns(d, P);
  for (int b = 0; b < d.B && order; ++b) {
    const int32_t* e = &P.blob[(size_t)b * P.stride];
    for (int k = 0; k < e[2]; ++k) order[e[3] + k] = e[1] + k;
  }
  return P.nF;
}

int tfm_layer_fwd(const tfm_dims* dims, const int32_t* n_train, const uint8_t* cell_mask,
                  const void* X, const float* params, void* Y, void* saved, size_t saved_bytes,
                  void* workspace, size_t workspace_bytes, void* stream) {
  Dims d;
  int rc = check_dims(dims, d);
  if (rc) return rc;
  if (!aligned(X) || !aligned(params) || !aligned(Y) || !aligned(saved) || !aligned(workspace))
    return fail(TFM_ERR_POINTER, "X, params, Y, saved and workspace must be non-null and "
                                 "16-byte aligned");
  const SavedLayout S = saved_layout(d);
  const WsLayout W = ws_layout(d);
  if (saved_bytes < saved_total(d))
    return fail(TFM_ERR_BUFFER, "saved buffer has %zu bytes, %zu required", saved_bytes,
                saved_total(d));
  if (workspace_bytes < W.total)
    return fail(TFM_ERR_BUFFER, "workspace has %zu bytes, %zu required", workspace_bytes,
                W.total);
  Plan P;
  rc = make_plan(d, n_train, cell_mask, P);
  if (rc) return rc;
  hipStream_t s = (hipStream_t)stream;
  char* ws = (char*)workspace;
  char* sv = (char*)saved;
  tfm::Geo g;
  const bool fast = fast_eligible(d);
  FastWs f{};
  tfm::SetupWeights sw{};
  if (fast) {
    f = fast_ws(d, ws, W);
    sw = setup_weights(d, params, f, false);
  }
  rc = setup_geo(d, P, ws, W.meta, g, fast ? &sw : nullptr, s);
  if (rc) return rc;
  if (d.block == TFM_BLOCK_PRENORM)
    return fwd_pre(d, g, (const tfm::bf16*)X, params, (tfm::bf16*)Y,
                   bufs_from_pre_saved(sv, pre_saved_layout(d)), f, s);
  if (d.dtype == TFM_F32)
    return fwd_simple<float>(d, g, (const float*)X, params, (float*)Y, sv, S, ws, W, s);
  if (fast)
    return fwd_fast(d, g, (const tfm::bf16*)X, params, (tfm::bf16*)Y, bufs_from_saved(sv, S), f,
                    s);
  return fwd_simple<tfm::bf16>(d, g, (const tfm::bf16*)X, params, (tfm::bf16*)Y, sv, S, ws, W,
                               s);
}

int tfm_layer_bwd(const tfm_dims* dims, const int32_t* n_train, const uint8_t* cell_mask,
                  const void* X, const float* params, const void* saved, size_t saved_bytes,
                  const void* dY, void* dX, float* grads, int accumulate, void* workspace,
                  size_t workspace_bytes, void* stream) {
  Dims d;
  int rc = check_dims(dims, d);
  if (rc) return rc;
  if (!aligned(X) || !aligned(params) || !aligned(saved) || !aligned(dY) || !aligned(dX) ||
      !aligned(grads) || !aligned(workspace))
    return fail(TFM_ERR_POINTER, "X, params, saved, dY, dX, grads and workspace must be "
                                 "non-null and 16-byte aligned");
  const SavedLayout S = saved_layout(d);
  const WsLayout W = ws_layout(d);
  if (saved_bytes < saved_total(d))
    return fail(TFM_ERR_BUFFER, "saved buffer has %zu bytes, %zu required", saved_bytes,
                saved_total(d));
  if (workspace_bytes < W.total)
    return fail(TFM_ERR_BUFFER, "workspace has %zu bytes, %zu required", workspace_bytes,
                W.total);
  Plan P;
  rc = make_plan(d, n_train, cell_mask, P);
  if (rc) return rc;
  hipStream_t s = (hipStream_t)stream;
  char* ws = (char*)workspace;
  tfm::Geo g;
  const bool fast = fast_eligible(d);
  tfm::SetupWeights sw{};
  if (fast) {
    order_columns(d, P);
    sw = setup_weights(d, params, fast_ws(d, ws, W), true);
  }
  rc = setup_geo(d, P, ws, W.meta, g, fast ? &sw : nullptr, s);
  if (rc) return rc;
  if (d.block == TFM_BLOCK_PRENORM)
    return bwd_pre(d, g, P, params, (const char*)saved, pre_saved_layout(d),
                   (const tfm::bf16*)dY, (tfm::bf16*)dX, grads, accumulate, ws, W, s);
  if (d.dtype == TFM_F32)
    return bwd_simple<float>(d, g, (const float*)X, params, (const char*)saved, S,
                             (const float*)dY, (float*)dX, grads, accumulate, ws, W, s);
  if (fast)
    return bwd_fast(d, g, P, (const tfm::bf16*)X, params, (const char*)saved, S,
                    (const tfm::bf16*)dY, (tfm::bf16*)dX, grads, accumulate, ws, W, s);
  return bwd_simple<tfm::bf16>(d, g, (const tfm::bf16*)X, params, (const char*)saved, S,
                               (const tfm::bf16*)dY, (tfm::bf16*)dX, grads, accumulate, ws, W,
                               s);
}

// Allocation-free forward: the plan and the bf16 weights in the library's static scratch.
int tfm_layer_fwd_noalloc(const tfm_dims* dims, const int32_t* n_train, const uint8_t* cell_mask,
                          const void* X, const float* params, void* Y, void* saved,
                          size_t saved_bytes, void* stream) {
  Dims d;
  int rc = check_dims(dims, d);
  if (rc) return rc;
  if (!infer_eligible(d))
    return fail(TFM_ERR_DIMS, "tfm_layer_fwd_noalloc needs TFM_BF16, E in {64, 128, 192, 256} "
                              "and H a multiple of E");
  if (!aligned(X) || !aligned(params) || !aligned(Y) || !aligned(saved))
    return fail(TFM_ERR_POINTER, "X, params, Y and saved must be non-null and 16-byte aligned");
  Arena a;
  const MetaOff M = take_meta(d, a);
  const tfm::WOff wo = tfm::weight_offsets(d.E, d.H);
  const size_t w_off = a.take((size_t)wo.total * 2);
  if (a.off > tfm::kStaticScratchBytes)
    return fail(TFM_ERR_BUFFER, "these dims need %zu bytes of library scratch; the maximum is "
                                "%zu (TFM_NOALLOC_SCRATCH_BYTES)", a.off,
                tfm::kStaticScratchBytes);
  if (saved_bytes < saved_total(d))
    return fail(TFM_ERR_BUFFER, "saved buffer has %zu bytes, %zu required", saved_bytes,
                saved_total(d));
  Plan P;
  rc = make_plan(d, n_train, cell_mask, P);
  if (rc) return rc;
  hipStream_t s = (hipStream_t)stream;
  void* base = nullptr;
  HIPCHK(tfm::static_scratch(s, &base));
  char* ws = (char*)base;
  FastWs f{};
  f.wo = wo;
  f.w = (tfm::bf16*)(ws + w_off);
  const tfm::SetupWeights sw = setup_weights(d, params, f, false);
  tfm::Geo g;
  rc = setup_geo(d, P, ws, M, g, &sw, s);
  if (rc) return rc;
  char* sv = (char*)saved;
  if (d.block == TFM_BLOCK_PRENORM)
    return fwd_pre(d, g, (const tfm::bf16*)X, params, (tfm::bf16*)Y,
                   bufs_from_pre_saved(sv, pre_saved_layout(d)), f, s);
  return fwd_fast(d, g, (const tfm::bf16*)X, params, (tfm::bf16*)Y,
                  bufs_from_saved(sv, saved_layout(d)), f, s);
}

// Shared checks of the thinking-row calls (the dims, the workspace that holds the column map,
// the plan from n_train and the mask, 1 <= T <= every n_train), then the column map upload.
static int thinking_setup(const tfm_dims* dims, const int32_t* n_train, const uint8_t* cell_mask,
                          int T, void* workspace, size_t workspace_bytes, Dims& d, tfm::Geo& g,
                          hipStream_t s) {
  int rc = check_dims(dims, d);
  if (rc) return rc;
  if (!aligned(workspace)) return fail(TFM_ERR_POINTER, "workspace must be 16-byte aligned");
  // only the column map is used: it leads both the training and the forward-only workspaces
  Arena a;
  const MetaOff M = take_meta(d, a);
  if (workspace_bytes < a.off)
    return fail(TFM_ERR_BUFFER, "workspace has %zu bytes, %zu required", workspace_bytes, a.off);
  Plan P;
  rc = make_plan(d, n_train, cell_mask, P);
  if (rc) return rc;
  for (int b = 0; b < d.B; ++b)
    if (T < 1 || T > n_train[b])
      return fail(TFM_ERR_DIMS, "T=%d thinking rows outside [1, n_train[%d]=%d]", T, b,
                  n_train[b]);
  return setup_geo(d, P, (char*)workspace, M, g, nullptr, s);
}

int tfm_thinking_rows_fwd(const tfm_dims* dims, const int32_t* n_train, const uint8_t* cell_mask,
                          int T, const float* table, void* X, void* workspace,
                          size_t workspace_bytes, void* stream) {
  Dims d;
  tfm::Geo g;
  hipStream_t s = (hipStream_t)stream;
  if (!aligned(table) || !aligned(X))
    return fail(TFM_ERR_POINTER, "table and X must be non-null and 16-byte aligned");
  int rc = thinking_setup(dims, n_train, cell_mask, T, workspace, workspace_bytes, d, g, s);
  if (rc) return rc;
  if (d.dtype == TFM_F32) HIPCHK(tfm::launch_thinking_fwd<float>(g, T, table, (float*)X, s));
  else HIPCHK(tfm::launch_thinking_fwd<tfm::bf16>(g, T, table, (tfm::bf16*)X, s));
  return TFM_OK;
}

int tfm_thinking_rows_bwd(const tfm_dims* dims, const int32_t* n_train, const uint8_t* cell_mask,
                          int T, const void* dX, float* dtable, int accumulate, void* workspace,
                          size_t workspace_bytes, void* stream) {
  Dims d;
  tfm::Geo g;
  hipStream_t s = (hipStream_t)stream;
  if (!aligned(dX) || !aligned(dtable))
    return fail(TFM_ERR_POINTER, "dX and dtable must be non-null and 16-byte aligned");
  int rc = thinking_setup(dims, n_train, cell_mask, T, workspace, workspace_bytes, d, g, s);
  if (rc) return rc;
  if (d.dtype == TFM_F32)
    HIPCHK(tfm::launch_thinking_bwd<float>(g, T, (const float*)dX, dtable, accumulate, s));
  else
    HIPCHK(tfm::launch_thinking_bwd<tfm::bf16>(g, T, (const tfm::bf16*)dX, dtable, accumulate,
                                               s));
  return TFM_OK;
}

size_t tfm_infer_workspace_bytes(const tfm_dims* dims) {
  Dims d;
  if (check_dims(dims, d) != TFM_OK) return 0;
  if (!infer_eligible(d)) {
    fail(TFM_ERR_DIMS, "forward-only calls need TFM_BF16, E in {64, 128, 192, 256} and H a "
                       "multiple of E");
    return 0;
  }
  return infer_layout(d).total;
}

size_t tfm_infer_cache_bytes(const tfm_dims* dims) {
  Dims d;
  if (check_dims(dims, d) != TFM_OK) return 0;
  return 2 * cache_half(d);
}

int tfm_layer_fwd_context(const tfm_dims* dims, const int32_t* n_train, const uint8_t* cell_mask,
                          const void* X, const float* params, void* Y, void* kv_cache,
                          size_t cache_bytes, void* workspace, size_t workspace_bytes,
                          void* stream) {
  return infer_call(dims, -1, n_train, cell_mask, X, params, Y, kv_cache, cache_bytes,
                    workspace, workspace_bytes, (hipStream_t)stream);
}

int tfm_layer_fwd_query(const tfm_dims* dims, int32_t context_rows, const int32_t* n_train,
                        const uint8_t* cell_mask, const void* X, const float* params,
                        const void* kv_cache, size_t cache_bytes, void* Y, void* workspace,
                        size_t workspace_bytes, void* stream) {
  if (context_rows < 0) return fail(TFM_ERR_DIMS, "context_rows=%d must be >= 1", context_rows);
  return infer_call(dims, context_rows, n_train, cell_mask, X, params, Y,
                    const_cast<void*>(kv_cache), cache_bytes, workspace, workspace_bytes,
                    (hipStream_t)stream);
}

}  // extern "C"
