// Launches of the bf16 MFMA attention kernels; included by one translation unit per form (attention.hip: whole tiles,
// attention_edge.hip: EDGE).
#pragma once
#include <hip/hip_runtime.h>

#include "attention.h"
#include "attention_mfma.h"

namespace varuna {

template <int D, bool DROP, bool EDGE>
inline hipError_t attn_fwd_mfma_d(const bf16* qkv, bf16* ctx, float* lse, int b, int s, int heads, int d, int causal,
                                  const DropArgs& drop, hipStream_t st) {
  const dim3 grid((unsigned)(heads * b), (unsigned)((s + 127) / 128));
  const float sl = 1.4426950408889634f / sqrtf((float)d);
  if (causal) hipLaunchKernelGGL((attn_fwd_mfma_kernel<D, true, DROP, EDGE>), grid, dim3(256), 0, st, qkv, ctx, lse, s, heads, sl, drop, d);
  else hipLaunchKernelGGL((attn_fwd_mfma_kernel<D, false, DROP, EDGE>), grid, dim3(256), 0, st, qkv, ctx, lse, s, heads, sl, drop, d);
  return hipGetLastError();
}

template <int D, bool DROP, bool EDGE>
inline hipError_t attn_bwd_mfma_d(const bf16* qkv, const bf16* ctx, const float* lse, const bf16* dctx, bf16* dqkv,
                                  float* delta, int b, int s, int heads, int d, int causal, const DropArgs& drop, hipStream_t st) {
  const dim3 grid((unsigned)(heads * b), (unsigned)((s + 127) / 128));
  const float sc = 1.0f / sqrtf((float)d), sl = 1.4426950408889634f * sc;
  if (causal) {
    hipLaunchKernelGGL((attn_bwd_dq_mfma_kernel<D, true, DROP, EDGE>), grid, dim3(256), 0, st, qkv, ctx, lse, dctx, dqkv, delta, s, heads, sc, sl, drop, d);
    hipLaunchKernelGGL((attn_bwd_dkv_mfma_kernel<D, true, DROP, EDGE>), grid, dim3(256), 0, st, qkv, lse, dctx, delta, dqkv, s, heads, sc, sl, drop, d);
  } else {
    hipLaunchKernelGGL((attn_bwd_dq_mfma_kernel<D, false, DROP, EDGE>), grid, dim3(256), 0, st, qkv, ctx, lse, dctx, dqkv, delta, s, heads, sc, sl, drop, d);
    hipLaunchKernelGGL((attn_bwd_dkv_mfma_kernel<D, false, DROP, EDGE>), grid, dim3(256), 0, st, qkv, lse, dctx, delta, dqkv, s, heads, sc, sl, drop, d);
  }
  return hipGetLastError();
}

template <int D, bool EDGE>
inline hipError_t attn_fwd_mfma(const bf16* qkv, bf16* ctx, float* lse, int b, int s, int heads, int d, int causal,
                                const DropArgs& drop, hipStream_t st) {
  return drop.thr != 0 ? attn_fwd_mfma_d<D, true, EDGE>(qkv, ctx, lse, b, s, heads, d, causal, drop, st)
                       : attn_fwd_mfma_d<D, false, EDGE>(qkv, ctx, lse, b, s, heads, d, causal, drop, st);
}

template <int D, bool EDGE>
inline hipError_t attn_bwd_mfma(const bf16* qkv, const bf16* ctx, const float* lse, const bf16* dctx, bf16* dqkv, float* delta,
                                int b, int s, int heads, int d, int causal, const DropArgs& drop, hipStream_t st) {
  return drop.thr != 0 ? attn_bwd_mfma_d<D, true, EDGE>(qkv, ctx, lse, dctx, dqkv, delta, b, s, heads, d, causal, drop, st)
                       : attn_bwd_mfma_d<D, false, EDGE>(qkv, ctx, lse, dctx, dqkv, delta, b, s, heads, d, causal, drop, st);
}

}  // namespace varuna
