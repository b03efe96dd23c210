#include "gemm_dma_launch.h"

namespace varuna {

hipError_t launch_gemm_dma_fwd(int mode, int variant, const bf16* a, int64_t lda, const bf16* b, int64_t ldb, int64_t M, int64_t N,
                                 int64_t K, const EpiArgs<bf16>& epi, hipStream_t st) {
  if (mode == EPI_BIAS) return dg_launch_variant<true, true, EPI_BIAS>(variant, a, lda, b, ldb, M, N, K, epi, 1, st);
  if (mode == EPI_BIAS_GELU) return dg_launch_variant<true, true, EPI_BIAS_GELU>(variant, a, lda, b, ldb, M, N, K, epi, 1, st);
  if (mode == EPI_BIAS_RES) return dg_launch_variant<true, true, EPI_BIAS_RES>(variant, a, lda, b, ldb, M, N, K, epi, 1, st);
  return hipErrorInvalidValue;
}

}  // namespace varuna
