#include "gemm_dma_launch.h"

namespace varuna {

hipError_t launch_gemm_dma_dgrad(int mode, int variant, const bf16* a, int64_t lda, const bf16* b, int64_t ldb, int64_t M, int64_t N,
                                 int64_t K, const EpiArgs<bf16>& epi, hipStream_t st) {
  if (mode == EPI_PLAIN) return dg_launch_variant<true, false, EPI_PLAIN>(variant, a, lda, b, ldb, M, N, K, epi, 1, st);
  if (mode == EPI_DGELU) return dg_launch_variant<true, false, EPI_DGELU>(variant, a, lda, b, ldb, M, N, K, epi, 1, st);
  return hipErrorInvalidValue;
}

}  // namespace varuna
