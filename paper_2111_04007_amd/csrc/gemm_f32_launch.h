// Launches of the GEMM kernels with fp32 products and on bf16 pieces; included by one translation unit per operand type.
#pragma once
#include <hip/hip_runtime.h>

#include "gemm_cut.h"
#include "gemm_f32.h"
#include "gemm_f32_few.h"

namespace varuna {

template <int MODE, bool AK, bool BK, int BM, int BN, int WM, int WN, int KS, int BKT>
inline hipError_t gf_launch_tile(bool vec, const float* a, int64_t lda, const float* b, int64_t ldb, int64_t M, int64_t N, int64_t K,
                                 const EpiArgs<float>& epi, hipStream_t st) {
  const int64_t tm = (M + BM - 1) / BM, tn = (N + BN - 1) / BN;
  if (tm > (1 << 27) || tn > (1 << 27) || tm * tn >= (1ll << 31)) return hipErrorInvalidValue;
  // a grid dimension holds less than 2^32 threads: 2^22 blocks of up to 512, then a second one (blocks past the last tile end)
  constexpr int64_t line = 1 << 22;
  const int64_t tiles = tm * tn;
  const dim3 grid((unsigned)(tiles < line ? tiles : line), (unsigned)((tiles + line - 1) / line)), block((BM / WM) * (BN / WN) * KS * kWave);
  if (vec) hipLaunchKernelGGL((gemm_f32_kernel<MODE, AK, BK, BM, BN, WM, WN, KS, BKT, true>), grid, block, 0, st, a, lda, b, ldb, M, N, K, (int)tm, (int)tn, epi);
  else hipLaunchKernelGGL((gemm_f32_kernel<MODE, AK, BK, BM, BN, WM, WN, KS, BKT, false>), grid, block, 0, st, a, lda, b, ldb, M, N, K, (int)tm, (int)tn, epi);
  return hipGetLastError();
}

template <typename T, int MODE, bool AK, bool BK, int TM, int TN, int KS>
inline hipError_t gc_launch(const T* a, int64_t lda, const T* b, int64_t ldb, int64_t M, int64_t N, int64_t K, const EpiArgs<T>& epi, hipStream_t st) {
  using G = GcTile<T, MODE, AK, BK, TM, TN, KS>;
  auto kern = gemm_cut_kernel<T, MODE, AK, BK, TM, TN, KS>;
  static const hipError_t attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)G::SMEM);
  if (attr_err != hipSuccess) return attr_err;
  const int64_t tm = (M + G::BM - 1) / G::BM, tn = (N + G::BN - 1) / G::BN, tiles = tm * tn;
  if (tm > (1 << 27) || tn > (1 << 27) || tiles >= (1ll << 31)) return hipErrorInvalidValue;
  constexpr int64_t line = 1 << 22;   // (a grid dimension as below)
  const dim3 grid((unsigned)(tiles < line ? tiles : line), (unsigned)((tiles + line - 1) / line));
  hipLaunchKernelGGL(kern, grid, dim3(G::NT), G::SMEM, st, a, lda, b, ldb, M, N, K, (int)tm, (int)tn, epi);
  return hipGetLastError();
}

template <bool BK, int MODE, bool LN>
inline hipError_t few_launch(const float* a, const float* b, int64_t M, int64_t N, int64_t K, const EpiArgs<float>& epi, const LnIn& ln, hipStream_t st) {
  const dim3 grid((unsigned)((N + 15) / 16), (unsigned)((M + 15) / 16)), block(kFewWaves * kWave);
  if (K <= 128) hipLaunchKernelGGL((gemm_f32_few_kernel<BK, MODE, 1, LN>), grid, block, 0, st, a, b, (int)M, (int)N, (int)K, epi, ln);
  else if (K <= 256) hipLaunchKernelGGL((gemm_f32_few_kernel<BK, MODE, 2, LN>), grid, block, 0, st, a, b, (int)M, (int)N, (int)K, epi, ln);
  else hipLaunchKernelGGL((gemm_f32_few_kernel<BK, MODE, 4, LN>), grid, block, 0, st, a, b, (int)M, (int)N, (int)K, epi, ln);
  return hipGetLastError();
}

template <typename T, int MODE, bool AK, bool BK>
inline hipError_t gf_launch(const T* a, int64_t lda, const T* b, int64_t ldb, int64_t M, int64_t N, int64_t K,
                            const EpiArgs<T>& epi, hipStream_t st) {
  const int64_t t32 = gf_tiles(M, N, 32), t64 = gf_tiles(M, N, 64);
  // whole pieces of four along the contiguous direction of both operands, from an aligned base
  const bool vec = ((reinterpret_cast<uintptr_t>(a) | reinterpret_cast<uintptr_t>(b)) & 15) == 0 && lda % 4 == 0 && ldb % 4 == 0;
  switch (gc_kind(sizeof(T) == 4, vec, AK && BK, t32, t64, K)) {
    case GC_32_8: return gc_launch<T, MODE, AK, BK, 1, 1, 8>(a, lda, b, ldb, M, N, K, epi, st);
    case GC_32_4: return gc_launch<T, MODE, AK, BK, 1, 1, 4>(a, lda, b, ldb, M, N, K, epi, st);
    case GC_64_4: return gc_launch<T, MODE, AK, BK, 2, 2, 4>(a, lda, b, ldb, M, N, K, epi, st);
    case GC_64_1: return gc_launch<T, MODE, AK, BK, 2, 2, 1>(a, lda, b, ldb, M, N, K, epi, st);
    case GC_NONE: break;
  }
  if constexpr (sizeof(T) == 4) {
    if constexpr (AK) {
      if (vec && gf_few(M, N, K)) return few_launch<BK, MODE, false>(a, b, M, N, K, epi, LnIn{}, st);
    }
    if (gf_small_tile(t32, t64)) return gf_launch_tile<MODE, AK, BK, 32, 32, 32, 32, 8, 128>(vec, a, lda, b, ldb, M, N, K, epi, st);
    return gf_launch_tile<MODE, AK, BK, 64, 64, 32, 32, 1, 64>(vec, a, lda, b, ldb, M, N, K, epi, st);
  }
  return hipErrorInvalidValue;
}

template <typename T>
hipError_t launch_gemm_f32(int op, int mode, const T* a, const T* b, int64_t M, int64_t N, int64_t K,
                                  const EpiArgs<T>& epi, hipStream_t st) {
  if (op == GEMM_FWD) {
    if (mode == EPI_BIAS) return gf_launch<T, EPI_BIAS, true, true>(a, K, b, K, M, N, K, epi, st);
    if (mode == EPI_BIAS_GELU) return gf_launch<T, EPI_BIAS_GELU, true, true>(a, K, b, K, M, N, K, epi, st);
    if (mode == EPI_BIAS_RES) return gf_launch<T, EPI_BIAS_RES, true, true>(a, K, b, K, M, N, K, epi, st);
  } else if (op == GEMM_DGRAD) {
    if (mode == EPI_PLAIN) return gf_launch<T, EPI_PLAIN, true, false>(a, K, b, N, M, N, K, epi, st);
    if (mode == EPI_DGELU) return gf_launch<T, EPI_DGELU, true, false>(a, K, b, N, M, N, K, epi, st);
  } else if (op == GEMM_WGRAD) {
    if (mode == EPI_ACCUM_F32) return gf_launch<T, EPI_ACCUM_F32, false, false>(a, M, b, N, M, N, K, epi, st);
  }
  return hipErrorInvalidValue;
}

// f(table, workgroups) for up to kMaxGroupJobs jobs at a time, tiles of BM x BN.
template <typename T, int BM, int BN, typename F>
inline hipError_t gf_for_groups(const WgradJob<T>* jobs, int n, int64_t K, F&& f) {
  for (int i0 = 0; i0 < n; i0 += kMaxGroupJobs) {
    GfGroup<T> g{};
    g.n = n - i0 < kMaxGroupJobs ? n - i0 : kMaxGroupJobs;
    g.K = K;
    int64_t blocks = 0;
    for (int i = 0; i < g.n; ++i) {
      g.job[i] = jobs[i0 + i];
      g.first[i] = (int)blocks;
      blocks += ((int64_t)((g.job[i].M + BM - 1) / BM) * ((g.job[i].N + BN - 1) / BN) + 7) / 8 * 8;
      if (blocks >= (1ll << 31)) return hipErrorInvalidValue;
    }
    g.first[g.n] = (int)blocks;
    f(g, (unsigned)blocks);
  }
  return hipGetLastError();
}
template <int BM, int BN, int WM, int WN, int KS, int BKT, bool VEC>
inline hipError_t gf_launch_group(const WgradJob<float>* jobs, int n, int64_t K, hipStream_t st) {
  return gf_for_groups<float, BM, BN>(jobs, n, K, [&](const GfGroup<float>& g, unsigned blocks) {
    hipLaunchKernelGGL((gemm_f32_group_kernel<BM, BN, WM, WN, KS, BKT, VEC>), dim3(blocks), dim3((BM / WM) * (BN / WN) * KS * kWave), 0, st, g);
  });
}
template <typename T, int TM, int TN, int KS>
inline hipError_t gc_launch_group(const WgradJob<T>* jobs, int n, int64_t K, hipStream_t st) {
  using G = GcTile<T, EPI_ACCUM_F32, false, false, TM, TN, KS>;
  auto kern = gemm_cut_group_kernel<T, TM, TN, KS>;
  static const hipError_t attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)G::SMEM);
  if (attr_err != hipSuccess) return attr_err;
  return gf_for_groups<T, G::BM, G::BN>(jobs, n, K, [&](const GfGroup<T>& g, unsigned blocks) {
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(G::NT), G::SMEM, st, g);
  });
}

}  // namespace varuna
