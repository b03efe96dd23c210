#include "gemm_f32_launch.h"

namespace varuna {

template hipError_t launch_gemm_f32<bf16>(int, int, const bf16*, const bf16*, int64_t, int64_t, int64_t, const EpiArgs<bf16>&, hipStream_t);

hipError_t launch_gemm_cut_group(const WgradJob<bf16>* jobs, int n, int64_t K, hipStream_t st) {
  int64_t t32 = 0;
  for (int i = 0; i < n; ++i) t32 += gf_tiles(jobs[i].M, jobs[i].N, 32);
  return t32 <= 512 ? gc_launch_group<bf16, 1, 1, 4>(jobs, n, K, st) : gc_launch_group<bf16, 2, 2, 4>(jobs, n, K, st);
}

}  // namespace varuna
