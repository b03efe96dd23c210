#include "gemm_dma_launch.h"

namespace varuna {

__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float* __restrict__ partial, int splits, int64_t n,
                                                            float* __restrict__ out) {
  const int64_t n4 = n / 4;  // n is a multiple of 4 (tile sizes)
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4; i += (int64_t)gridDim.x * blockDim.x) {
    floatx4 acc = reinterpret_cast<floatx4*>(out)[i];
    for (int s = 0; s < splits; ++s) {
      const floatx4 p = reinterpret_cast<const floatx4*>(partial + (int64_t)s * n)[i];
      acc[0] += p[0]; acc[1] += p[1]; acc[2] += p[2]; acc[3] += p[3];
    }
    reinterpret_cast<floatx4*>(out)[i] = acc;
  }
}

hipError_t launch_splitk_reduce(const float* partial, int splits, int64_t n, float* out, hipStream_t st) {
  int64_t nblk = (n / 4 + 255) / 256;
  if (nblk > 8192) nblk = 8192;
  if (nblk < 1) nblk = 1;
  hipLaunchKernelGGL(splitk_reduce_kernel, dim3((unsigned)nblk), dim3(256), 0, st, partial, splits, n, out);
  return hipGetLastError();
}

hipError_t launch_gemm_dma_wgrad(int mode, int variant, const bf16* a, int64_t lda, const bf16* b, int64_t ldb, int64_t M, int64_t N,
                                 int64_t K, const EpiArgs<bf16>& epi, hipStream_t st, int splits) {
  if (mode == EPI_ACCUM_F32) return dg_launch_variant<false, false, EPI_ACCUM_F32>(variant, a, lda, b, ldb, M, N, K, epi, splits, st);
  if (mode == EPI_STORE_F32) return dg_launch_variant<false, false, EPI_STORE_F32>(variant, a, lda, b, ldb, M, N, K, epi, splits, st);
  if (mode == EPI_PLAIN) return dg_launch_variant<false, false, EPI_PLAIN>(variant, a, lda, b, ldb, M, N, K, epi, splits, st);
  return hipErrorInvalidValue;
}

}  // namespace varuna
