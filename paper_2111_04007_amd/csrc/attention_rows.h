// One row of attention on one wave, without LDS: what the tiled kernels fall back to for a row whose tiled result is not
// finite.  A tile multiplies its masked entries with weight zero, which lets an infinity or NaN of a masked token (0 * inf)
// into rows that must not see it, and a running maximum of -inf (a tile whose scores are all -inf) makes the rescale NaN.
// Here a row reads only the tokens its mask admits, and the softmax takes its maximum over all of them first.
// A lane owns keys (forward, dQ) or queries (dK, dV) lane + 64 c and columns lane and lane + 64: d <= 128.
#pragma once
#include "common.h"

namespace varuna {

// The lane, read anew: like the shuffles below it shares nothing with the code before, whose loops have no register to keep
// a lane number or shuffle address in for these rare rows.
__device__ __forceinline__ int ar_lane() {
  int lane;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(lane));
  return lane;
}
__device__ __forceinline__ float ar_xor(float v, int o, int lane) {
  return __int_as_float(__builtin_amdgcn_ds_bpermute((lane ^ o) << 2, __float_as_int(v)));
}
__device__ __forceinline__ float ar_sum(float v, int lane) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += ar_xor(v, o, lane);
  return v;
}
__device__ __forceinline__ float ar_max(float v, int lane) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, ar_xor(v, o, lane));
  return v;
}

// Whether x is an infinity or NaN adds NaN to the sum; finite values leave it as it is.
__device__ __forceinline__ float ar_probe(float sum, float x) { return fmaf(x, 0.f, sum); }
// Rows (lane % 32 of the wave's 32) whose probe sum is not finite, from either half of the wave.
__device__ __forceinline__ uint32_t ar_bad_rows(float probe) {
  const uint64_t b = __ballot(!(probe == 0.f));
  return (uint32_t)b | (uint32_t)(b >> 32);
}

// f(e) for every element of a row, in the order in which the fp32 matrix products add them (attention_f32.h: k-values 8g + i, then
// 8g + 4 + i, one fma each).  A score is then the same to the bit in either form.  It has to be: the rounding of a long score is in
// the forward's log-sum-exp as well, and cancels in the backward's probability only if both computed the same (rows peaked on
// one key, forward on one form and backward on the other: twice the error of dV).  bf16 rows, whose results are rounded to 2^-9, keep
// the plain order, which their loads like better (2-5 % of the backward).
template <typename T, typename F>
__device__ __forceinline__ void ar_elements(int d, F&& f) {
  if constexpr (sizeof(T) == 2) {
    for (int e = 0; e < d; ++e) f(e);
    return;
  }
  int e = 0;
  for (; e + 8 <= d; e += 8) {
#pragma unroll
    for (int i = 0; i < 4; ++i) { f(e + i); f(e + 4 + i); }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (e + i < d) f(e + i);
    if (e + 4 + i < d) f(e + 4 + i);
  }
}
template <typename T>
__device__ __forceinline__ float ar_dot(const T* __restrict__ a, const T* __restrict__ b, int d) {
  float dot = 0.f;
  ar_elements<T>(d, [&](int e) { dot = fmaf(to_f32(a[e]), to_f32(b[e]), dot); });
  return dot;
}

// acc{0,1} += sum over n <= 64 rows of w (held by lane j for row j) * base[j * ld + {lane, lane + 64}]
template <typename T>
__device__ __forceinline__ void ar_weighted(float& acc0, float& acc1, const T* __restrict__ base, int64_t ld, int n, float w, int d, int lane) {
  for (int j = 0; j < n; ++j) {
    const float wj = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(w), j));
    if (lane < d) acc0 = fmaf(wj, to_f32(base[j * ld + lane]), acc0);
    if (lane + 64 < d) acc1 = fmaf(wj, to_f32(base[j * ld + lane + 64]), acc1);
  }
}
template <typename T>
__device__ __forceinline__ void ar_store(T* __restrict__ row, float v0, float v1, int d, int lane) {
  if (lane < d) row[lane] = from_f32<T>(v0);
  if (lane + 64 < d) row[lane + 64] = from_f32<T>(v1);
}

// ctx and log-sum-exp (lse may be null) of query i; base: the head's Q columns of the first token of its sequence, h columns
// to its K and to its V; ctx: its context columns; stat: index of (batch, head, first token) in lse and the mask's rows.
template <typename T>
__device__ __forceinline__ void ar_fwd(const T* __restrict__ base, T* __restrict__ ctx, float* __restrict__ lse, int i, int s, int h, int d,
                                       bool causal, float scale, int64_t stat, const DropArgs& drop, int lane) {
  const int64_t ld = 3 * (int64_t)h;
  const T *q = base + i * ld, *k = base + h, *v = k + h;
  const int nk = causal ? i + 1 : s;
  float mx = -INFINITY;
  for (int key = lane; key < nk; key += kWave) mx = fmaxf(mx, ar_dot(q, k + key * ld, d) * scale);
  mx = ar_max(mx, lane);
  float sum = 0.f, a0 = 0.f, a1 = 0.f;
  for (int k0 = 0; k0 < nk; k0 += kWave) {
    const int key = k0 + lane;
    float p = 0.f;
    if (key < nk) {
      p = expf(ar_dot(q, k + key * ld, d) * scale - mx);
      sum += p;   // the softmax is normalised before the dropout
      if (drop.thr != 0 && !drop_keep(drop, drop_row_word(drop, (uint32_t)(stat + i), (uint32_t)key >> 2), key & 3)) p = 0.f;
    }
    ar_weighted(a0, a1, v + k0 * ld, ld, nk - k0 < kWave ? nk - k0 : kWave, p, d, lane);
  }
  sum = ar_sum(sum, lane);
  const float inv = (drop.thr != 0 ? drop.scale : 1.0f) / sum;
  if (lse && lane == 0) lse[stat + i] = mx + logf(sum);
  ar_store(ctx + (int64_t)i * h, a0 * inv, a1 * inv, d, lane);
}

// dQ of query i; ctx, dctx and dq: the head's columns of the first token (rows of h, h and 3h).
template <typename T>
__device__ __forceinline__ void ar_dq(const T* __restrict__ base, const T* __restrict__ ctx, const T* __restrict__ dctx, const float* __restrict__ lse,
                                      T* __restrict__ dqkv, int i, int s, int h, int d, bool causal, float scale, int64_t stat,
                                      const DropArgs& drop, int lane) {
  const int64_t ld = 3 * (int64_t)h;
  const T *q = base + i * ld, *k = base + h, *v = k + h, *g = dctx + (int64_t)i * h, *o = ctx + (int64_t)i * h;
  float dl = 0.f;
  for (int e = lane; e < d; e += kWave) dl += to_f32(g[e]) * to_f32(o[e]);
  dl = ar_sum(dl, lane);
  const float l = lse[stat + i];
  const int nk = causal ? i + 1 : s;
  float a0 = 0.f, a1 = 0.f;
  for (int k0 = 0; k0 < nk; k0 += kWave) {
    const int key = k0 + lane;
    float ds = 0.f;
    if (key < nk) {
      float dp = ar_dot(g, v + key * ld, d);
      if (drop.thr != 0)
        dp = drop_keep(drop, drop_row_word(drop, (uint32_t)(stat + i), (uint32_t)key >> 2), key & 3) ? dp * drop.scale : 0.f;
      ds = expf(ar_dot(q, k + key * ld, d) * scale - l) * (dp - dl);
    }
    ar_weighted(a0, a1, k + k0 * ld, ld, nk - k0 < kWave ? nk - k0 : kWave, ds, d, lane);
  }
  ar_store(dqkv + i * ld, a0 * scale, a1 * scale, d, lane);
}

// dK and dV of key `key`; dqkv: the head's Q columns of the first token, as in base.  ctx: null, or where delta is not in place yet, the head's
// context columns it is summed from.
template <typename T>
__device__ __forceinline__ void ar_dkv(const T* __restrict__ base, const T* __restrict__ dctx, const float* __restrict__ lse,
                                       const float* __restrict__ delta, T* __restrict__ dqkv, int key, int s, int h, int d, bool causal,
                                       float scale, int64_t stat, const DropArgs& drop, int lane, const T* __restrict__ ctx = nullptr) {
  const int64_t ld = 3 * (int64_t)h;
  const T *k = base + h + key * ld, *v = k + h;
  float k0_ = 0.f, k1_ = 0.f, v0_ = 0.f, v1_ = 0.f;
  for (int i0 = causal ? key : 0; i0 < s; i0 += kWave) {
    const int i = i0 + lane;
    float pp = 0.f, ds = 0.f;
    if (i < s) {
      const float pr = expf(ar_dot(base + i * ld, k, d) * scale - lse[stat + i]);
      float f = 1.0f;
      if (drop.thr != 0) f = drop_keep(drop, drop_row_word(drop, (uint32_t)(stat + i), (uint32_t)key >> 2), key & 3) ? drop.scale : 0.f;
      pp = pr * f;
      const float dl = ctx ? ar_dot(dctx + (int64_t)i * h, ctx + (int64_t)i * h, d) : delta[stat + i];
      ds = pr * (ar_dot(dctx + (int64_t)i * h, v, d) * f - dl);
    }
    const int n = s - i0 < kWave ? s - i0 : kWave;
    ar_weighted(k0_, k1_, base + i0 * ld, ld, n, ds, d, lane);
    ar_weighted(v0_, v1_, dctx + (int64_t)i0 * h, h, n, pp, d, lane);
  }
  ar_store(dqkv + key * ld + h, k0_ * scale, k1_ * scale, d, lane);
  ar_store(dqkv + key * ld + 2 * h, v0_, v1_, d, lane);
}

}  // namespace varuna
