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
// Whether a call ends sooner with one wave per row than with fp32 products, whose waves work through whole 32x32 tiles however few
// there are (and load element by element where `vec`, whole pieces of four from an aligned base, does not hold).  Rows are
// many small tasks, so what counts is their work rows * s * d; long rows are a chain each, which the other form cuts into tiles.
// Limits by operand type, loads, direction and padded head dim {32, 64, 96, 128}: longest row, work in 2^20; set on 2650 shapes (d
// 7 .. 128, s 4 .. 512, 1 .. 256 heads), where the choice is within 6 % of the better form on 98 in 100.  us, per row / fp32
// products, forward and backward: fp32 8 heads of 128 over 64 tokens 10.5 / 16.3 and 36 / 50, 256 heads 90 / 32 and 394 / 103; 4
// heads of 99 over 48 8.0 / 22.8 and 25 / 86; bf16 16 heads of 100 over 32 7.3 / 13.1 and 17 / 46, 32 heads of 35 over 128
// 20.2 / 14.6 and 70 / 49.  (fp32 forwards of up to 1024 rows of 32 tokens: equal alone, per row sooner inside a step.)
inline bool attn_rows_sooner(bool f32, bool vec, bool backward, int b, int s, int heads, int d) {
  struct Limit { int s, work; };
  constexpr Limit limit[2][2][2][4] = {
      {{{{0, 0}, {192, 6}, {192, 9}, {192, 19}}, {{64, 1}, {192, 11}, {96, 13}, {192, 26}}},      // bf16, single elements
       {{{0, 0}, {0, 0}, {64, 13}, {64, 16}}, {{48, 2}, {64, 9}, {64, 13}, {96, 16}}}},           // bf16, pieces
      {{{{0, 0}, {256, 14}, {512, 19}, {512, 46}}, {{64, 1}, {256, 14}, {256, 19}, {512, 46}}},   // fp32, single elements
       {{{0, 0}, {0, 0}, {64, 7}, {192, 18}}, {{64, 2}, {64, 5}, {64, 7}, {80, 10}}}}};           // fp32, pieces
  const int64_t rows = (int64_t)b * heads * s;
  if (f32 && !backward && s <= 32 && rows <= 1024) return true;
  const Limit& l = limit[f32][vec][backward][(d + 31) / 32 - 1];
  return s <= l.s && rows * s * d <= (int64_t)l.work << 20;
}
// Whole pieces of four elements from an aligned base: rows start at multiples of d.
template <typename T>
inline bool attn_f32_vec(const void* p, const void* q, const void* r, int d) {
  return d % 4 == 0 && ((reinterpret_cast<uintptr_t>(p) | reinterpret_cast<uintptr_t>(q) | reinterpret_cast<uintptr_t>(r)) & (4 * sizeof(T) - 1)) == 0;
}
template <typename T>
hipError_t launch_attention_fwd_f32(const T* qkv, T* ctx, float* lse, int b, int s, int heads, int d, int causal,
                                    const DropArgs& drop, hipStream_t st);
template <typename T>
hipError_t launch_attention_bwd_f32(const T* qkv, const T* ctx, const float* lse, const T* dctx, T* dqkv, float* delta, int b,
                                    int s, int heads, int d, int causal, const DropArgs& drop, hipStream_t st);

// fp32 in tiles of 16 (attention_f32_16.h): head dims up to 128 in whole 16-byte pieces (the tensors must be 16-byte aligned).
inline bool attn_f32_16_supported(int d) { return d % 4 == 0 && d <= 128; }
// Whether a call they take ends sooner with one wave per row: rows of a few tokens leave most of a tile empty, which counts where the tiles take more
// than one round (2 to 4 workgroups a CU forward, 4 to 1 backward), and one or two tokens also within one.  Longest row by padded head dim {32, 64, 96, 128}: with any
// number of heads, with more than p1, with more than p2; set on 1900 shapes (d 16 .. 128, s 1 .. 192, 1 .. 16384 heads), where the choice is within 8 % of the better
// form on 99 in 100.  us, per row / tiles of 16, forward and backward: one token, 4096 heads of 128 8.7 / 31, 24 / 166, of 64 6.6 / 12.7, 15 / 52, 16 heads of 128
// 5.1 / 5.5, 6.8 / 7.7; four tokens, 1024 heads of 128 9.2 / 9.6, 25 / 45, 128 heads 5.8 / 5.4, 9.3 / 7.7; 192 tokens, 1 head of 128 26 / 10, 71 / 22.
// The smallest calls (up to 128 rows, 512 above d = 64) that go to the row kernels rather than to tiles of 32 do so here as well, which is no matter of speed (2
// heads of 64 over 64 tokens 7.3 / 4.5, 14.3 / 6.8; 8 of 128 over 64 10.7 / 6.1, 26 / 10.8): test_short_rows_go_to_the_row_kernels holds such calls to
// those kernels' bits.
inline bool attn_f32_16_rows(bool backward, int b, int s, int heads, int d) {
  struct Limit { int any, p1, s1, p2, s2; };
  constexpr Limit limit[2][4] = {{{0, 1024, 2, 1024, 2}, {0, 1024, 3, 1024, 3}, {0, 768, 3, 768, 3}, {2, 512, 4, 512, 4}},
                                 {{1, 1535, 3, 1535, 3}, {2, 767, 4, 767, 4}, {2, 128, 4, 767, 8}, {2, 128, 4, 767, 8}}};
  const Limit& l = limit[backward][(d + 31) / 32 - 1];
  const int64_t pairs = (int64_t)b * heads;
  if (pairs * s <= (d <= 64 ? 128 : 512) && attn_rows_sooner(true, true, backward, b, s, heads, d)) return true;
  return s <= (pairs > l.p2 ? l.s2 : pairs > l.p1 ? l.s1 : l.any);
}
// Whether the other calls they take go there.  Against tiles of 32: half the rows per workgroup, so twice as many workgroups with half a chain each, for twice
// the operand traffic per product.  Set on 2051 shapes (d 32 .. 128, s 192 .. 4096, 4 .. 1024 heads), where the choice is within 6 % of the better form on
// 99 in 100.  us, tiles of 32 / of 16:
//   d above 64: sooner forward (32 heads of 128 over 1000 causal 273 / 127, 64 of 96 over 1000 full 581 / 338) and backward (64 of 96 over 1000 1797 / 1476, 128 of 128
//     over 1000 7116 / 5042), except backward at d = 128 unmasked in equal rounds of 256 workgroups with few rows and heads (24 of 128 over 1000 913 / 943).
//   d up to 64, forward: sooner by the shorter chains (24 of 64 over 500 causal 25 / 19, full 34 / 27) while an XCD's L2 serves the second reading.  Workgroups go to
//     the eight XCDs in turn, heads first, so one XCD works on pairs / gcd(pairs, 8) heads side by side; the more there are, the shorter rows must be (35 heads of 64
//     over 840 tokens causal 64 / 58, 1664 175 / 217; 78 over 600 full 109 / 128; 256 over 512 full 243 / 300).  Unmasked rows above 320 only in fewer rounds; at d = 32
//     long rows are no shorter (32 heads over 3000 tokens causal 239 / 259).
//   d up to 64, backward: sooner up to several 100000 rows (128 of 64 over 1000 causal 1040 / 920, 1024 over 512 full 4351 / 4973).
inline bool attn_f32_16(bool backward, int b, int s, int heads, int d, bool causal) {
  const int64_t pairs = (int64_t)b * heads, rows = pairs * s;
  const int64_t rounds16 = (pairs * ((s + 15) / 16) + 255) / 256, rounds32 = (pairs * ((s + 31) / 32) + 255) / 256;
  const int64_t heads_per_xcd = pairs / (pairs % 8 == 0 ? 8 : pairs % 4 == 0 ? 4 : pairs % 2 == 0 ? 2 : 1);
  if (backward) {
    if (d <= 32) return rows <= (causal ? 700000 : 550000);
    if (d <= 64) return rows <= (causal ? 520000 : 350000);
    return d <= 96 || causal || s <= 320 || rounds16 < 2 * rounds32 || rows >= 65000 || heads_per_xcd > 25;
  }
  if (d > 64) return true;
  if (causal && d <= 32) return pairs <= 8 || (rows * s <= 64000000 && (heads_per_xcd <= 45 || s <= 400));
  if (causal) return heads_per_xcd <= 16 || s <= (heads_per_xcd <= 25 ? 1600 : heads_per_xcd <= 45 ? 700 : 350);
  if (s <= 224 || (s <= 320 && heads_per_xcd <= (d <= 32 ? 75 : 45))) return true;
  return heads_per_xcd <= (s <= 900 ? 25 : 16) && (d <= 32 ? 1.06 : 1.0) * (double)rounds16 < 2.0 * (double)rounds32;
}
hipError_t launch_attention_fwd_f32_16(const float* qkv, float* ctx, float* lse, int b, int s, int heads, int d, int causal, const DropArgs& drop, hipStream_t st);
hipError_t launch_attention_bwd_f32_16(const float* qkv, const float* ctx, const float* lse, const float* dctx, float* dqkv, float* delta, int b, int s,
                                        int heads, int d, int causal, const DropArgs& drop, hipStream_t st);

template <typename T>
hipError_t launch_attention_fwd_simple(const T* qkv, T* ctx, float* lse, int b, int s, int heads, int d, int causal,
                                       const DropArgs& drop, hipStream_t st);
template <typename T>
hipError_t launch_attention_bwd_simple(const T* qkv, const T* ctx, const float* lse, const T* dctx, T* dqkv, float* delta, int b,
                                       int s, int heads, int d, int causal, const DropArgs& drop, hipStream_t st);

}  // namespace varuna
