#include "gemm_f32_launch.h"

namespace varuna {

template hipError_t launch_gemm_f32<float>(int, int, const float*, const float*, int64_t, int64_t, int64_t, const EpiArgs<float>&, hipStream_t);

bool ln_gemm_f32_takes(const float* b, const LnIn& ln, int64_t M, int64_t N, int64_t K) {
  const void* p[] = {b, ln.gamma, ln.beta, ln.y, ln.copy};   // (a: buffer loads, which take any float's address)
  for (const void* q : p)
    if ((reinterpret_cast<uintptr_t>(q) & 15) != 0) return false;
  return K % 4 == 0 && K <= 512 && gf_few(M, N, K);
}
hipError_t launch_ln_gemm_f32(int mode, const float* a, const float* b, int64_t M, int64_t N, int64_t K, const EpiArgs<float>& epi, const LnIn& ln, hipStream_t st) {
  if (mode == EPI_BIAS) return few_launch<true, EPI_BIAS, true>(a, b, M, N, K, epi, ln, st);
  if (mode == EPI_BIAS_GELU) return few_launch<true, EPI_BIAS_GELU, true>(a, b, M, N, K, epi, ln, st);
  return hipErrorInvalidValue;
}

// Odd rows: from 128 tokens on as launch_gemm_cut_group, below in fp32 products (gc_kind).  Micro-batches of whole steps (us, 32x32 on 4
// waves / 64x64 on 4 / 64x64 on 1 / fp32 products): 66 wide over 2048 tokens 279 / 293 / 352 / 299, 258 wide (783 tiles) over 512 401 / 413 / 414 / 453, 390 wide
// (2041) over 8192 2180 / 2169 / 2220 / 3401, 774 wide (7250) over 512 895 / 892 / 849 / 1131.
hipError_t launch_gemm_f32_group(const WgradJob<float>* jobs, int n, int64_t K, hipStream_t st) {
  int64_t t32 = 0, t64 = 0;
  bool vec = true;
  for (int i = 0; i < n; ++i) {
    t32 += gf_tiles(jobs[i].M, jobs[i].N, 32);
    t64 += gf_tiles(jobs[i].M, jobs[i].N, 64);
    vec = vec && ((reinterpret_cast<uintptr_t>(jobs[i].a) | reinterpret_cast<uintptr_t>(jobs[i].b)) & 15) == 0 && jobs[i].M % 4 == 0 && jobs[i].N % 4 == 0;
  }
  if (!vec && K >= 128) return t32 <= 512 ? gc_launch_group<float, 1, 1, 4>(jobs, n, K, st) : gc_launch_group<float, 2, 2, 4>(jobs, n, K, st);
  if (gf_small_tile(t32, t64))
    return vec ? gf_launch_group<32, 32, 32, 32, 8, 128, true>(jobs, n, K, st) : gf_launch_group<32, 32, 32, 32, 8, 128, false>(jobs, n, K, st);
  return vec ? gf_launch_group<64, 64, 32, 32, 1, 64, true>(jobs, n, K, st) : gf_launch_group<64, 64, 32, 32, 1, 64, false>(jobs, n, K, st);
}

}  // namespace varuna
