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

template <typename T>
hipError_t launch_attention_fwd_simple(const T* qkv, T* ctx, float* lse, int b, int s, int heads, int d, int causal,
                                       const DropArgs& drop, hipStream_t st);
template <typename T>
hipError_t launch_attention_bwd_simple(const T* qkv, const T* ctx, const float* lse, const T* dctx, T* dqkv, float* delta, int b,
                                       int s, int heads, int d, int causal, const DropArgs& drop, hipStream_t st);

}  // namespace varuna
