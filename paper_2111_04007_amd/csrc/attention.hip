#include "attention_launch.h"
#include "attention_simple.h"

namespace varuna {

hipError_t launch_attention_fwd_mfma(const bf16* qkv, bf16* ctx, float* lse, int b, int s, int heads, int d, int causal,
                                     const DropArgs& drop, hipStream_t st) {
  if (d == 64) return attn_fwd_mfma<64, false>(qkv, ctx, lse, b, s, heads, d, causal, drop, st);
  if (d == 96) return attn_fwd_mfma<96, false>(qkv, ctx, lse, b, s, heads, d, causal, drop, st);
  if (d == 128) return attn_fwd_mfma<128, false>(qkv, ctx, lse, b, s, heads, d, causal, drop, st);
  return hipErrorInvalidConfiguration;
}

hipError_t launch_attention_bwd_mfma(const bf16* qkv, const bf16* ctx, const float* lse, const bf16* dctx, bf16* dqkv,
                                     float* delta, int b, int s, int heads, int d, int causal, const DropArgs& drop, hipStream_t st) {
  if (d == 64) return attn_bwd_mfma<64, false>(qkv, ctx, lse, dctx, dqkv, delta, b, s, heads, d, causal, drop, st);
  if (d == 96) return attn_bwd_mfma<96, false>(qkv, ctx, lse, dctx, dqkv, delta, b, s, heads, d, causal, drop, st);
  if (d == 128) return attn_bwd_mfma<128, false>(qkv, ctx, lse, dctx, dqkv, delta, b, s, heads, d, causal, drop, st);
  return hipErrorInvalidConfiguration;
}

}  // namespace varuna
