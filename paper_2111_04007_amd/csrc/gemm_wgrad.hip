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

template <int BM, int BN, int WGM, int WGN, bool EDGE>
static hipError_t group_launch(const DgJob* jobs, int n, int64_t K, hipStream_t st) {
  auto kern = gemm_group_kernel<BM, BN, WGM, WGN, EDGE>;
  constexpr size_t smem = dg_smem_bytes<BM, BN, WGM, WGN, EPI_ACCUM_F32, 4>();
  static const hipError_t attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                         hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  if (attr_err != hipSuccess) return attr_err;
  for (int i0 = 0; i0 < n; i0 += kMaxGroupJobs) {
    DgGroup g{};
    g.n = n - i0 < kMaxGroupJobs ? n - i0 : kMaxGroupJobs;
    g.K = (int)K;
    int64_t blocks = 0;
    for (int i = 0; i < g.n; ++i) {
      g.job[i] = jobs[i0 + i];
      g.first[i] = (int)blocks;
      const int64_t tiles = (int64_t)((g.job[i].M + BM - 1) / BM) * ((g.job[i].N + BN - 1) / BN);
      blocks += (tiles + 7) / 8 * 8;
      if (blocks >= (1ll << 31)) return hipErrorInvalidValue;
    }
    g.first[g.n] = (int)blocks;
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(WGM * WGN * kWave), smem, st, g, 8);
  }
  return hipGetLastError();
}

hipError_t launch_gemm_group(int variant, const DgJob* jobs, int n, int64_t K, hipStream_t st) {
  switch (variant) {
    case 18: return group_launch<256, 256, 2, 4, false>(jobs, n, K, st);
    case 19: return group_launch<128, 128, 2, 2, false>(jobs, n, K, st);
    case 22: return group_launch<128, 128, 2, 2, true>(jobs, n, K, st);
    case 23: return group_launch<256, 256, 2, 4, true>(jobs, n, K, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_gemm_dma_wgrad(int mode, int variant, const bf16* a, int64_t lda, const bf16* b, int64_t ldb, int64_t M, int64_t N,
                                 int64_t K, const EpiArgs<bf16>& epi, hipStream_t st, int splits) {
  if (mode == EPI_ACCUM_F32) return dg_launch_variant<false, false, EPI_ACCUM_F32>(variant, a, lda, b, ldb, M, N, K, epi, splits, st);
  if (mode == EPI_STORE_F32) return dg_launch_variant<false, false, EPI_STORE_F32>(variant, a, lda, b, ldb, M, N, K, epi, splits, st);
  if (mode == EPI_PLAIN) return dg_launch_variant<false, false, EPI_PLAIN>(variant, a, lda, b, ldb, M, N, K, epi, splits, st);
  return hipErrorInvalidValue;
}

}  // namespace varuna
