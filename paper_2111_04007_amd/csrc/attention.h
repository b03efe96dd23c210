// What the stage needs of the attention kernels: the shapes they take and their launches (attention.hip).
// qkv is [b*s, 3h] (Q | K | V column blocks, head j at column j*d of each), ctx / dctx are [b*s, h],
// lse / delta are [b, heads, s] fp32.
#pragma once
#include "common.h"

namespace varuna {

constexpr int ATS_MAX_S = 4096;
constexpr int ATS_MAX_D = 256;

inline bool attn_mfma_supported(int s, int d) { return (d == 64 || d == 96 || d == 128) && s >= 128 && s % 128 == 0; }
// What the EDGE form takes: rows of a head that are whole 16-byte pieces (the tensors must be 16-byte aligned).
inline bool attn_edge_supported(int d) { return d % 8 == 0 && d <= 128; }

hipError_t launch_attention_fwd_mfma(const bf16* qkv, bf16* ctx, float* lse, int b, int s, int heads, int d, int causal,
                                     const DropArgs& drop, hipStream_t st);
hipError_t launch_attention_bwd_mfma(const bf16* qkv, const bf16* ctx, const float* lse, const bf16* dctx, bf16* dqkv,
                                     float* delta, int b, int s, int heads, int d, int causal, const DropArgs& drop, hipStream_t st);

// The EDGE forms (attention_edge.hip).
hipError_t launch_attention_fwd_mfma_edge(const bf16* qkv, bf16* ctx, float* lse, int b, int s, int heads, int d, int causal,
                                     const DropArgs& drop, hipStream_t st);
hipError_t launch_attention_bwd_mfma_edge(const bf16* qkv, const bf16* ctx, const float* lse, const bf16* dctx, bf16* dqkv,
                                     float* delta, int b, int s, int heads, int d, int causal, const DropArgs& drop, hipStream_t st);

// The tiled forms take (batch, head) as one grid dimension of 256-thread blocks, and a dimension holds less than 2^32 threads;
// beyond, the per-row kernels (three dimensions) serve.
inline bool attn_grid_ok(int b, int heads) { return (int64_t)b * heads < (1ll << 24); }
// fp32 products on the matrix cores (attention_f32.h), head dims up to 128.
inline bool attn_f32_supported(int d) { return d <= 128; }
// A call of a few short rows ends sooner with one wave per row: a wave of the other form works through whole 32x32 tiles, 7-8 us
// forward and 20-25 us backward for any call that leaves the chip idle.  Measured (us forward / backward, per row against
// fp32 products; batch x length x heads x dim): 2x32x2x64 5.2 / 12 against 7.3 / 22, 2x64x2x64 6.8 / 19 against 7.8 / 23
// (forward inside a step, operands out of cache: 9.7 against 8.0), 1x32x16x64 5.2 / 12 against 7.4 / 22; but 2x96x2x64 9.1 /
// 29 against 8.2 / 24, 8x32x16x64 9.5 / 31 against 7.4 / 23.
inline bool attn_few_rows(int b, int s, int heads, bool backward) {
  return s <= (backward ? 64 : 32) && (int64_t)b * heads * s <= 1024;
}
template <typename T>
hipError_t launch_attention_fwd_f32(const T* qkv, T* ctx, float* lse, int b, int s, int heads, int d, int causal,
                                    const DropArgs& drop, hipStream_t st);
template <typename T>
hipError_t launch_attention_bwd_f32(const T* qkv, const T* ctx, const float* lse, const T* dctx, T* dqkv, float* delta, int b,
                                    int s, int heads, int d, int causal, const DropArgs& drop, hipStream_t st);

template <typename T>
hipError_t launch_attention_fwd_simple(const T* qkv, T* ctx, float* lse, int b, int s, int heads, int d, int causal,
                                       const DropArgs& drop, hipStream_t st);
template <typename T>
hipError_t launch_attention_bwd_simple(const T* qkv, const T* ctx, const float* lse, const T* dctx, T* dqkv, float* delta, int b,
                                       int s, int heads, int d, int causal, const DropArgs& drop, hipStream_t st);

}  // namespace varuna
