// fp32 products of few output elements (gf_few: at most 512 tiles of 16x16, more of short sums; less than 1024 k): out = A B^T or A B with fp32 products (v_mfma_f32_16x16x4_f32), A [M,K]
// k-major, whole 16-byte pieces.  One workgroup of 8 waves per 16x16 tile; a wave takes every eighth 16 k.
//
// What bounds such a product is latency: a launch, one way to memory, the sums' way through LDS.  So there is no staging: a wave's
// operands, up to 64 k of both, go straight into registers in one batch, or two above 512 k (a lane holds k-values 16u + 4*(lane/16) .. +3 of row lane%16 of its
// unit u, the products take them in the same order on both sides), what the epilogue reads is fetched with them, and the only barrier is the
// one where the eight sums meet.  Tiles of 16x16 rather than 32x32: four times as many workgroups, each with half as much
// to load (64 KB at K = 512, 0.4 us of a CU's path from L2).
//
// LN: A is the layer norm of x, whose statistics the workgroup takes from its own registers on the way (two more barriers); the workgroups of the
// first tile column store the normalised rows, the statistics and a copy of x where they are wanted.  K up to 512: the rows stay in registers.
#pragma once
#include "common.h"
#include "gemm_f32.h"

namespace varuna {

constexpr int kFewWaves = 8;   // waves per tile

// Units of 16 k of one operand, from buffer loads: k past the end of the reduction reads as zero.
template <bool KMAJOR, int U>
struct FewLoader {
  floatx4 v[U];
  const float* base;
  uint32_t extent, row;   // bytes of the operand; of the lane's row (k-major) or column
  int ld;
  __device__ __forceinline__ void init(const float* p, int64_t rows, int K, int i) {
    base = p;
    extent = (uint32_t)(rows * K * 4);
    ld = KMAJOR ? K : (int)rows;
    row = (uint32_t)i * (KMAJOR ? (uint32_t)K * 4 : 4u);
  }
  __device__ __forceinline__ void load(int u0, int quad, int K) {
#if defined(__HIP_DEVICE_COMPILE__)  // the buffer builtins exist in the device pass only
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), 0, extent, 0x00020000);
#pragma unroll
    for (int j = 0; j < U; ++j) {
      const int k = (u0 + kFewWaves * j) * 16 + 4 * quad;   // (K is a multiple of 4)
      if constexpr (KMAJOR) {
        v[j] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)(k < K ? row + (uint32_t)k * 4 : 0xfffffff0u), 0, 0));
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          v[j][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)(k < K ? row + (uint32_t)(k + e) * (uint32_t)ld * 4 : 0xfffffff0u), 0, 0));
      }
    }
#endif
  }
};

template <bool BK, int MODE, int U, bool LN>
__global__ __launch_bounds__(kFewWaves* kWave) void gemm_f32_few_kernel(const float* __restrict__ a, const float* __restrict__ b, int M, int N, int K,
                                                                        EpiArgs<float> epi, LnIn ln) {
  __shared__ float red[kFewWaves][256];
  __shared__ float part[LN ? 2 : 1][kFewWaves][16];
  const int tid = threadIdx.x, lane = tid % kWave, i16 = lane & 15, quad = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int m0 = blockIdx.y * 16, n0 = blockIdx.x * 16;
  const int m = m0 + i16 < M ? m0 + i16 : M - 1, n = n0 + i16 < N ? n0 + i16 : N - 1;   // rows past the end repeat the last one
  const int units = (K + 15) / 16;
  FewLoader<true, U> fa;
  FewLoader<BK, U> fb;
  fa.init(a, M, K, m);
  fb.init(b, N, K, n);
  fa.load(wave, quad, K);
  floatx4 fg[LN ? U : 1], fs[LN ? U : 1];
  if constexpr (LN) {
#pragma unroll
    for (int j = 0; j < U; ++j) {
      const int k = (wave + kFewWaves * j) * 16 + 4 * quad, kk = k < K ? k : 0;
      fg[j] = *reinterpret_cast<const floatx4*>(ln.gamma + kk);
      fs[j] = *reinterpret_cast<const floatx4*>(ln.beta + kk);
    }
  }
  fb.load(wave, quad, K);
  // Thread t < 256 finishes element t of the tile: row 4 * (t % 64 / 16) + t / 64, column t % 16.
  const int om = m0 + 4 * quad + wave, on = n0 + i16;
  float bias = 0.f, old = 0.f;
  if (wave < 4) {
    bias = epilogue_bias<float, MODE>(epi, n);
    old = epilogue_fetch<float, MODE>(epi, om < M ? om : M - 1, n);
  }
  __builtin_amdgcn_sched_barrier(0);   // everything is on its way before the first wait

  if constexpr (LN) {
    // mean, then the centred second moment, as in norm_reduce.h
    auto row_sum = [&](float s, int which) {
      s += __shfl_xor(s, 16, kWave);
      s += __shfl_xor(s, 32, kWave);
      if (quad == 0) part[which][wave][i16] = s;
      __syncthreads();
      float t = 0.f;
#pragma unroll
      for (int w = 0; w < kFewWaves; ++w) t += part[which][w][i16];
      return t;
    };
    const bool store = blockIdx.x == 0 && m0 + i16 < M;
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < U; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) s += fa.v[j][e];
    const float mean = row_sum(s, 0) / (float)K;
    s = 0.f;
#pragma unroll
    for (int j = 0; j < U; ++j) {
      const int k = (wave + kFewWaves * j) * 16 + 4 * quad;
      if (k < K && store && ln.copy) *reinterpret_cast<floatx4*>(ln.copy + (int64_t)m * K + k) = fa.v[j];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        fa.v[j][e] = k < K ? fa.v[j][e] - mean : 0.f;
        s += fa.v[j][e] * fa.v[j][e];
      }
    }
    const float rstd = 1.0f / sqrtf(row_sum(s, 1) / (float)K + ln.eps);
#pragma unroll
    for (int j = 0; j < U; ++j) {
      const int k = (wave + kFewWaves * j) * 16 + 4 * quad;
#pragma unroll
      for (int e = 0; e < 4; ++e) fa.v[j][e] = k < K ? fg[j][e] * (fa.v[j][e] * rstd) + fs[j][e] : 0.f;
      if (k < K && store && ln.y) *reinterpret_cast<floatx4*>(ln.y + (int64_t)m * K + k) = fa.v[j];
    }
    if (store && ln.stats && tid < 16) { ln.stats[m] = mean; ln.stats[M + m] = rstd; }
  }

  floatx4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
  auto products = [&](const floatx4 (&x)[U], const floatx4 (&y)[U]) {
#pragma unroll
    for (int j = 0; j < U; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[j & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[j][e], y[j][e], acc[j & 1], 0, 0, 0);
  };
  bool more = false;
  if constexpr (!LN && U == 4) {   // more than 512 k: the others in flight during the products of these
    more = wave + kFewWaves * U < units;
    if (more) {
      auto na = fa;
      auto nb = fb;
      na.load(wave + kFewWaves * U, quad, K);
      nb.load(wave + kFewWaves * U, quad, K);
      __builtin_amdgcn_sched_barrier(0);
      products(fa.v, fb.v);
      products(na.v, nb.v);
    }
  }
  if (!more) products(fa.v, fb.v);
#pragma unroll
  for (int r = 0; r < 4; ++r) red[wave][r * 64 + lane] = acc[0][r] + acc[1][r];
  __syncthreads();
  if (wave >= 4 || om >= M || on >= N) return;
  float v = 0.f;
#pragma unroll
  for (int w = 0; w < kFewWaves; ++w) v += red[w][tid];
  epilogue_store<float, MODE>(epi, om, on, v, bias, old);
}

}  // namespace varuna
