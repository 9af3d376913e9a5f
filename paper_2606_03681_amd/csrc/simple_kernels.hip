// Small kernels: uploads through kernel arguments, column sums of the decoder's bias gradients.
#include "kernels.h"

namespace tfm {

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

// ============================================================================ column sums
__global__ void k_colsum(int64_t M, int Nj, const float* __restrict__ A, int64_t lda,
                         int64_t chunk, float* __restrict__ part) {
  int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= Nj) return;
  int64_t mb = (int64_t)blockIdx.y * chunk;
  int64_t me = (mb + chunk < M) ? mb + chunk : M;
  float acc = 0.f;
  for (int64_t m = mb; m < me; ++m) acc += A[m * lda + j];
  part[(int64_t)blockIdx.y * Nj + j] = acc;
}

hipError_t launch_colsum(int64_t M, int Nj, const float* A, int64_t lda, int64_t chunk,
                         float* partial, hipStream_t s) {
  int64_t Z = (M + chunk - 1) / chunk;
  if (Z < 1) Z = 1;
  dim3 grid((unsigned)((Nj + 255) / 256), (unsigned)Z);
  k_colsum<<<grid, 256, 0, s>>>(M, Nj, A, lda, chunk, partial);
  return hipGetLastError();
}

}  // namespace tfm
