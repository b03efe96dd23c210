#include "gemm_f32_launch.h"

namespace varuna {

template hipError_t launch_gemm_f32<bf16>(int, int, const bf16*, const bf16*, int64_t, int64_t, int64_t, const EpiArgs<bf16>&, hipStream_t);

// 32x32 tiles up to two rounds of them, where 64x64 would leave CUs idle, else 64x64; four waves each.  Micro-batches of whole steps
// (us, 32x32 on 8 waves / on 4 / 64x64 on 4 / on 1): 64 wide over 2048 tokens 120 / 120 / 129 / 149, 192 wide (432 tiles) over 2048 162 / 159 / 163 /
// 182, 256 wide (768) over 512 136 / 134 / 132 / 139 and over 8192 307 / 298 / 282 / 363, 384 wide (1728) over 64 125 / 118 / 117 / 114 and
// over 8192 492 / 470 / 429 / 472.
hipError_t launch_gemm_cut_group(const WgradJob<bf16>* jobs, int n, int64_t K, hipStream_t st) {
  int64_t t32 = 0;
  for (int i = 0; i < n; ++i) t32 += gf_tiles(jobs[i].M, jobs[i].N, 32);
  return t32 <= 512 ? gc_launch_group<bf16, 1, 1, 4>(jobs, n, K, st) : gc_launch_group<bf16, 2, 2, 4>(jobs, n, K, st);
}

}  // namespace varuna
