// The one launch in front of every layer call: the device copy of the active-cell plan and the
// bf16 weights the call's products read.
#pragma once

#include "fast.h"

namespace tfm {

// Ints of the plan blob that travel as kernel arguments (longer blobs are uploaded first).
constexpr int SETUP_BLOB = 512;

struct SetupPlan {
  int32_t B, R, S, words;
  // per dataset: n_train, first active column, active columns, its first place in cord, mask words
  const int32_t* blob;  // host, B * (4 + words)
  DsInfo* ds;
  int32_t *dblob, *colmap, *col_ntr, *cord;
  int64_t* col_cell0;
};

// Weight forms a call needs.  Bit k of w / wt: matrix k of (Wqkv_f, Wo_f, Wqkv_i, Wo_i, W1, W2)
// as stored / transposed; fold: Wqkv_i and W1 in w carry the LayerNorm scale of their input and
// the folded biases are written; stream: 1 the fused MLP forward's weight stream, 2 the
// backward's.
struct SetupWeights {
  const float* params;
  int32_t E, H;
  uint32_t w, wt;
  int32_t fold, stream;
  WFold f;
  bf16 *wout, *wtout;
};

// wt null (no matrices): the plan alone.
hipError_t launch_setup(const SetupPlan& p, const SetupWeights* w, hipStream_t s);

}  // namespace tfm
