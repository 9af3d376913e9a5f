// Host-side launchers of the HIP kernels.  Each returns the hipError_t of its launch(es).
#pragma once

#include "common.h"

namespace tfm {

// ---- metadata -------------------------------------------------------------------------------
// Copies `count` int32 values from host memory into device memory at `dst` through kernel
// arguments (stream-ordered, no host synchronisation, host memory free to reuse at return).
hipError_t launch_upload(const int32_t* host, int64_t count, int32_t* dst, hipStream_t s);

// partial[z][j] = sum over rows m of chunk z of A[m * lda + j]
hipError_t launch_colsum(int64_t M, int Nj, const float* A, int64_t lda, int64_t chunk,
                         float* partial, hipStream_t s);

}  // namespace tfm
