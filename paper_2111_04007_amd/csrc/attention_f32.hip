#include <hip/hip_runtime.h>

#include "attention_f32.h"
#include "attention_f32_16.h"

namespace varuna {

template hipError_t launch_attention_fwd_f32<float>(const float*, float*, float*, int, int, int, int, int, const DropArgs&, hipStream_t);
template hipError_t launch_attention_bwd_f32<float>(const float*, const float*, const float*, const float*, float*, float*, int, int, int, int, int,
                                                  const DropArgs&, hipStream_t);

#define VARUNA_AW(KERNEL) \
  if (d <= 32) hipLaunchKernelGGL((KERNEL<32>), grid, block, 0, st, a, scale); \
  else if (d <= 64) hipLaunchKernelGGL((KERNEL<64>), grid, block, 0, st, a, scale); \
  else if (d <= 96) hipLaunchKernelGGL((KERNEL<96>), grid, block, 0, st, a, scale); \
  else hipLaunchKernelGGL((KERNEL<128>), grid, block, 0, st, a, scale); \
  return hipGetLastError();
hipError_t launch_attention_fwd_f32_16(const float* qkv, float* ctx, float* lse, int b, int s, int heads, int d, int causal, const DropArgs& drop, hipStream_t st) {
  const dim3 grid((unsigned)(heads * b), (unsigned)((s + 15) / 16)), block(AW_WAVES * kWave);
  const AwArgs a{qkv, ctx, lse, nullptr, nullptr, nullptr, s, heads, d, causal, drop};
  const float scale = 1.0f / sqrtf((float)d);
  VARUNA_AW(attn_f32_16_fwd_kernel)
}
hipError_t launch_attention_bwd_f32_16(const float* qkv, const float* ctx, const float* lse, const float* dctx, float* dqkv, float* delta, int b, int s,
                                       int heads, int d, int causal, const DropArgs& drop, hipStream_t st) {
  const dim3 grid((unsigned)(heads * b), (unsigned)(2 * ((s + 15) / 16))), block(AW_WAVES * kWave);
  const AwArgs a{qkv, const_cast<float*>(ctx), const_cast<float*>(lse), dctx, dqkv, delta, s, heads, d, causal, drop};
  const float scale = 1.0f / sqrtf((float)d);
  VARUNA_AW(attn_f32_16_bwd_kernel)
}
#undef VARUNA_AW

}  // namespace varuna
