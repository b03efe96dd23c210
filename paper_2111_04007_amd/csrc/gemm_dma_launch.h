// Launches of the bf16 MFMA GEMM kernels; included by one translation unit per product (gemm_fwd.hip, gemm_dgrad.hip,
// gemm_wgrad.hip), which are compiled side by side.
#pragma once
#include <hip/hip_runtime.h>

#include "gemm_dma.h"

namespace varuna {

template <int BM, int BN, int WGM, int WGN, bool AK, bool BK_, int MODE, int LS = 0, bool EDGE = false>
inline hipError_t dg_launch_one(const bf16* a, int64_t lda, const bf16* b, int64_t ldb, int64_t M, int64_t N,
                                int64_t K, const EpiArgs<bf16>& epi, int splits, hipStream_t st) {
  auto kern = gemm_dma_kernel<BM, BN, WGM, WGN, AK, BK_, MODE, LS, EDGE>;
  constexpr size_t smem = dg_smem_bytes<BM, BN, WGM, WGN, MODE, LS>();
  static_assert(smem <= 160 * 1024, "one workgroup's LDS");
  // the first call raises the kernel's dynamic LDS limit (thread-safe: initialisation of a local static)
  static const hipError_t attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                         hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  if (attr_err != hipSuccess) return attr_err;
  const int tm = (int)((M + BM - 1) / BM), tn = (int)((N + BN - 1) / BN);
  constexpr int xcd_remap = 1, group = 8;   // tile order: contiguous range per XCD, walked in groups of 8 tile rows
  if (splits < 1 || (MODE != EPI_STORE_F32 && splits != 1) || (K + DG_BK - 1) / DG_BK < splits) return hipErrorInvalidValue;
  hipLaunchKernelGGL(kern, dim3((unsigned)(tm * tn), (unsigned)splits), dim3(WGM * WGN * kWave), smem, st, a, lda, b, ldb,
                     (int)K, tm, tn, epi, xcd_remap, group, M, N);
  return hipGetLastError();
}

template <bool AK, bool BK_, int MODE>
inline hipError_t dg_launch_variant(int variant, const bf16* a, int64_t lda, const bf16* b, int64_t ldb,
                                    int64_t M, int64_t N, int64_t K, const EpiArgs<bf16>& epi, int splits, hipStream_t st) {
  switch (variant) {
    case 5: return dg_launch_one<256, 256, 2, 4, AK, BK_, MODE>(a, lda, b, ldb, M, N, K, epi, splits, st);
    case 6: return dg_launch_one<256, 256, 2, 2, AK, BK_, MODE>(a, lda, b, ldb, M, N, K, epi, splits, st);
    case 7: return dg_launch_one<128, 128, 2, 2, AK, BK_, MODE>(a, lda, b, ldb, M, N, K, epi, splits, st);
    case 8: return dg_launch_one<256, 128, 2, 2, AK, BK_, MODE>(a, lda, b, ldb, M, N, K, epi, splits, st);
    case 9: return dg_launch_one<256, 256, 2, 4, AK, BK_, MODE, 1>(a, lda, b, ldb, M, N, K, epi, splits, st);
    case 10: return dg_launch_one<128, 128, 2, 2, AK, BK_, MODE, 1>(a, lda, b, ldb, M, N, K, epi, splits, st);
    case 11: return dg_launch_one<256, 256, 2, 2, AK, BK_, MODE, 1>(a, lda, b, ldb, M, N, K, epi, splits, st);
    case 12: return dg_launch_one<256, 256, 2, 4, AK, BK_, MODE, 2>(a, lda, b, ldb, M, N, K, epi, splits, st);
    case 13: return dg_launch_one<256, 256, 2, 2, AK, BK_, MODE, 2>(a, lda, b, ldb, M, N, K, epi, splits, st);
    case 14: return dg_launch_one<128, 128, 2, 2, AK, BK_, MODE, 2>(a, lda, b, ldb, M, N, K, epi, splits, st);
    case 15: return dg_launch_one<128, 256, 2, 4, AK, BK_, MODE, 2>(a, lda, b, ldb, M, N, K, epi, splits, st);
    case 16: return dg_launch_one<256, 128, 4, 2, AK, BK_, MODE, 2>(a, lda, b, ldb, M, N, K, epi, splits, st);
    case 17: return dg_launch_one<256, 256, 2, 2, AK, BK_, MODE, 4>(a, lda, b, ldb, M, N, K, epi, splits, st);
    case 18: return dg_launch_one<256, 256, 2, 4, AK, BK_, MODE, 4>(a, lda, b, ldb, M, N, K, epi, splits, st);
    case 19: return dg_launch_one<128, 128, 2, 2, AK, BK_, MODE, 4>(a, lda, b, ldb, M, N, K, epi, splits, st);
    case 20: return dg_launch_one<128, 256, 2, 2, AK, BK_, MODE, 5>(a, lda, b, ldb, M, N, K, epi, splits, st);
    case 21: return dg_launch_one<256, 128, 2, 2, AK, BK_, MODE, 5>(a, lda, b, ldb, M, N, K, epi, splits, st);
    case 22: return dg_launch_one<128, 128, 2, 2, AK, BK_, MODE, 4, true>(a, lda, b, ldb, M, N, K, epi, splits, st);
    case 23: return dg_launch_one<256, 256, 2, 4, AK, BK_, MODE, 4, true>(a, lda, b, ldb, M, N, K, epi, splits, st);
    case 24:
      if constexpr (AK && BK_) return dg_launch_one<128, 192, 2, 2, AK, BK_, MODE, 5>(a, lda, b, ldb, M, N, K, epi, splits, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace varuna
