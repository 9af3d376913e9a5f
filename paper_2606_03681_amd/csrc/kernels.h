// Host-side launchers of the HIP kernels.  Each returns the hipError_t of its launch(es).
#pragma once

#include "common.h"

namespace tfm {

// ---- metadata -------------------------------------------------------------------------------
// Copies `count` int32 values from host memory into device memory at `dst` through kernel
// arguments (stream-ordered, no host synchronisation, host memory free to reuse at return).
hipError_t launch_upload(const int32_t* host, int64_t count, int32_t* dst, hipStream_t s);
// Expands the per-dataset blob {n_train, col0, S_b, mask words...} into DsInfo and the
// column maps of Geo.
hipError_t launch_expand_meta(const int32_t* blob, int B, int R, int S, int words, DsInfo* ds,
                              int32_t* col_ds, int32_t* col_c, int32_t* colmap,
                              int64_t* col_cell0, int32_t* col_ntr, hipStream_t s);

// ---- simple (VALU, fp32 arithmetic) kernels, any storage type ------------------------------
// partial[z][j] = sum over rows m of chunk z of A[m*lda+j] (* B[m*ldb+j] if B non-null)
template <class T>
hipError_t launch_colsum(int64_t M, int Nj, const T* A, int64_t lda, const T* B, int64_t ldb,
                         int64_t chunk, float* partial, hipStream_t s);
}  // namespace tfm
