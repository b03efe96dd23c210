#include "attention_launch.h"

namespace varuna {

hipError_t launch_attention_fwd_mfma_edge(const bf16* qkv, bf16* ctx, float* lse, int b, int s, int heads, int d, int causal,
                                     const DropArgs& drop, hipStream_t st) {
  if (d <= 32) return attn_fwd_mfma<32, true>(qkv, ctx, lse, b, s, heads, d, causal, drop, st);
  if (d <= 64) return attn_fwd_mfma<64, true>(qkv, ctx, lse, b, s, heads, d, causal, drop, st);
  if (d <= 96) return attn_fwd_mfma<96, true>(qkv, ctx, lse, b, s, heads, d, causal, drop, st);
  if (d <= 128) return attn_fwd_mfma<128, true>(qkv, ctx, lse, b, s, heads, d, causal, drop, st);
  return hipErrorInvalidConfiguration;
}

hipError_t launch_attention_bwd_mfma_edge(const bf16* qkv, const bf16* ctx, const float* lse, const bf16* dctx, bf16* dqkv,
                                     float* delta, int b, int s, int heads, int d, int causal, const DropArgs& drop, hipStream_t st) {
  if (d <= 32) return attn_bwd_mfma<32, true>(qkv, ctx, lse, dctx, dqkv, delta, b, s, heads, d, causal, drop, st);
  if (d <= 64) return attn_bwd_mfma<64, true>(qkv, ctx, lse, dctx, dqkv, delta, b, s, heads, d, causal, drop, st);
  if (d <= 96) return attn_bwd_mfma<96, true>(qkv, ctx, lse, dctx, dqkv, delta, b, s, heads, d, causal, drop, st);
  if (d <= 128) return attn_bwd_mfma<128, true>(qkv, ctx, lse, dctx, dqkv, delta, b, s, heads, d, causal, drop, st);
  return hipErrorInvalidConfiguration;
}

}  // namespace varuna
