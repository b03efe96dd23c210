// Softmax attention with fp32 products on the matrix cores (v_mfma_f32_32x32x2_f32): the fp32 path, and the bf16 shapes
// the bf16 MFMA kernels do not take (head dims that are no multiple of 8, tensors off a 16-byte boundary).  Head dim
// d up to 128 (padded to D in {32, 64, 96, 128} with zeros), any sequence length; no atomics.
//
// One workgroup of 4 waves per 32 queries (forward, dQ) or 32 keys (dK, dV) of one head; the waves take every fourth
// 32-row tile of the other side and their partial results are combined through LDS in a fixed order at the end.  A
// 32x32x2 product keeps a SIMD's matrix pipe for 64 clocks, so operands come straight from global memory into
// registers, with no LDS in the loop: a row operand as 16 bytes per lane of 32 rows (k-values 8g + 4*half + i for product
// i of group g), and the other operand of the second product as rows of 32 consecutive columns.  Scores are computed with
// the softmax row as the result's column, so a lane holds 16 scores of one row (query 8*(r/4) + 4*half + r%4 of
// register r in the key-side kernel, key in the others), and register r is the second product's operand as it stands.
//
// What bounds it: the fp32 matrix rate once the chip is full, the serial products of one wave below that.  Measured against the
// one-wave-per-row kernels (us; 2 x 500 tokens, 12 heads of 64, causal): forward 153 -> 26, backward 643 -> 82.
//
// A block that holds a result that is not finite works its rows out again one by one (attention_rows.h): what a masked token's
// infinity or NaN did to rows that must not see it is undone.  The check takes 0.1 - 0.2 us of a kernel.
#pragma once
#include "attention.h"
#include "attention_rows.h"
#include "common.h"

namespace varuna {

// e^x.  Its argument is a score minus a maximum or log-sum-exp in one rounding (the fma), with the factor log2(e) only then: folded
// into the scale it would add its rounding to the whole score, and another one to the log-sum-exp (up to twice the error of
// dV where softmax rows are peaked).
__device__ __forceinline__ float af_exp(float x) { return __builtin_amdgcn_exp2f(x * 1.4426950408889634f); }

// k-values 8g + 4*half .. +3 of one row of d columns for every group g; zeros past the end of the row.  (Here and below what
// lies outside is loaded from an element inside and replaced, so that no branch keeps a load from going out early.)
template <typename T, int D, bool VEC>
__device__ __forceinline__ void af_row(floatx4 (&f)[D / 8], const T* __restrict__ row, int half, int d) {
  typedef T Tx4 __attribute__((ext_vector_type(4)));
#pragma unroll
  for (int g = 0; g < D / 8; ++g) {
    const int e = 8 * g + 4 * half;
    floatx4 x;
    if constexpr (VEC) {
      const Tx4 t = *reinterpret_cast<const Tx4*>(row + (e < d ? e : 0));
#pragma unroll
      for (int i = 0; i < 4; ++i) x[i] = e < d ? to_f32((T)t[i]) : 0.f;
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float v = to_f32(row[e + i < d ? e + i : 0]);
        x[i] = e + i < d ? v : 0.f;
      }
    }
    f[g] = x;
  }
}

// acc[row of a][row of b] += sum over the head dim
template <int D>
__device__ __forceinline__ floatx16 af_dot(const floatx4 (&a)[D / 8], const floatx4 (&b)[D / 8]) {
  floatx16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
  for (int g = 0; g < D / 8; ++g)
#pragma unroll
    for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[g][i], b[g][i], acc, 0, 0, 0);
  return acc;
}

// Rows row0 + 8*(r/4) + 4*half + r%4 of a tile, columns db*32 + lane%32; zeros in rows past the end (columns past the end only
// reach results that are not stored).
template <typename T>
__device__ __forceinline__ void af_cols(float (&x)[16], const T* __restrict__ base, int64_t ld, int row0, int rows, int db, int d, int half, int l32) {
  const int col = db * 32 + l32 < d ? db * 32 + l32 : 0;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int row = row0 + 8 * (r >> 2) + 4 * half + (r & 3);
    const float v = to_f32(base[(int64_t)(row < rows ? row : rows - 1) * ld + col]);
    x[r] = row < rows ? v : 0.f;
  }
}
// acc[db][column of the tile][lane] += sum over the tile's 32 rows, weight w[r] for the lane's column of the result.  BUFS blocks of 32
// columns of the tile are held at a time: all of them, read ahead of the scores (af_ahead), up to D = 64; above, registers
// allow one, or two with the next one on its way during the products of one.  Taken by measurement (backward, us, against one
// block): D = 96 all three in dQ 68.6 -> 62.4 (4 heads of 72, 200 tokens), D = 128 two in both 308 -> 285 (2 heads, 1000 tokens);
// two blocks in the forward at D = 96 17.7 -> 21.8.
template <int D, int BUFS = D / 32> struct AfTile { float x[BUFS][16]; };
template <typename T, int D, int BUFS>
__device__ __forceinline__ void af_ahead(AfTile<D, BUFS>& t, const T* __restrict__ base, int64_t ld, int row0, int rows, int d, int half, int l32) {
  if constexpr (BUFS == D / 32) {
#pragma unroll
    for (int db = 0; db < D / 32; ++db) af_cols<T>(t.x[db], base, ld, row0, rows, db, d, half, l32);
    __builtin_amdgcn_sched_barrier(0);
  }
}
template <typename T, int D, int BUFS>
__device__ __forceinline__ void af_weighted(floatx16 (&acc)[D / 32], AfTile<D, BUFS>& t, const T* __restrict__ base, int64_t ld, int row0, int rows,
                                            int d, const floatx16& w, int half, int l32) {
  constexpr bool AHEAD = BUFS == D / 32;
  if constexpr (!AHEAD && BUFS == 2) af_cols<T>(t.x[0], base, ld, row0, rows, 0, d, half, l32);
#pragma unroll
  for (int db = 0; db < D / 32; ++db) {
    if constexpr (!AHEAD && BUFS == 1) af_cols<T>(t.x[0], base, ld, row0, rows, db, d, half, l32);
    if constexpr (!AHEAD && BUFS == 2) {
      if (db + 1 < D / 32) af_cols<T>(t.x[(db + 1) & 1], base, ld, row0, rows, db + 1, d, half, l32);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(t.x[AHEAD ? db : db % BUFS][r], w[r], acc[db], 0, 0, 0);
  }
}

template <int D> __device__ __forceinline__ void af_zero(floatx16 (&acc)[D / 32]) {
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[db][r] = 0.f;
}

constexpr int AF_WAVES = 4;
// Partial results [wave][lane's column][D + 4] in LDS: acc[db][r] is element db*32 + 8*(r/4) + 4*half + r%4 of column l32.
template <int D>
__device__ __forceinline__ void af_put(float* sm, const floatx16 (&acc)[D / 32], int wave, int half, int l32) {
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const floatx4 v = {acc[db][4 * g], acc[db][4 * g + 1], acc[db][4 * g + 2], acc[db][4 * g + 3]};
      *reinterpret_cast<floatx4*>(sm + (wave * 32 + l32) * (D + 4) + db * 32 + 8 * g + 4 * half) = v;
    }
}
template <int D>
__device__ __forceinline__ float af_get_sum(const float* sm, int row, int e) {
  float v = 0.f;
#pragma unroll
  for (int w = 0; w < AF_WAVES; ++w) v += sm[(w * 32 + row) * (D + 4) + e];
  return v;
}

// Arguments of the three kernels (the forward uses no dctx, dqkv and delta; the key side no ctx).
template <typename T>
struct AfArgs {
  const T* qkv; T* ctx; float* lse;
  const T* dctx; T* dqkv; float* delta;
  int s, heads, d, causal;
  DropArgs drop;
};
// Whether any thread of the block saw a result that is not finite (probe: ar_probe over what it stored); pad: the four unused words
// behind a row of the partial results.
__device__ __forceinline__ bool af_any(float* pad, float probe, int wave) {
  const float mine = __ballot(!(probe == 0.f)) != 0 ? 1.f : 0.f;
  if (ar_lane() == 0) pad[wave] = mine;
  __syncthreads();
  const floatx4 all = *reinterpret_cast<const floatx4*>(pad);
  return __builtin_amdgcn_readfirstlane(all[0] + all[1] + all[2] + all[3] != 0.f);
}
// f(arguments, row, lane, first element of its head in qkv and in ctx, its index in the statistics) for the block's 32 rows, shared
// out over the waves (attention_rows.h).  Everything is read anew from the argument segment: kept from the kernel's start for
// this rare path it would cost the loops their registers.
template <typename T, typename F>
__device__ __forceinline__ void af_rows(int block, int wave, F&& f) {
  auto seg = (const __attribute__((address_space(4))) AfArgs<T>*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(seg));
  const AfArgs<T> a = *(const AfArgs<T>*)seg;
  const int lane = ar_lane();
  const int64_t head = blockIdx.x % a.heads, bi = blockIdx.x / a.heads, tok = bi * a.s * a.heads * a.d;
  __threadfence();   // the results stored so far are in place in every wave before they are stored again
  __syncthreads();
  for (int row = block * 32 + wave; row < block * 32 + 32 && row < a.s; row += AF_WAVES)
    f(a, row, lane, 3 * tok + head * a.d, tok + head * a.d, (bi * a.heads + head) * a.s);
}

// ctx and log-sum-exp (lse may be null).
template <typename T, int D, bool VEC>
__global__ __launch_bounds__(AF_WAVES* kWave) void attn_f32_fwd_kernel(AfArgs<T> args, float scale) {
  const T* __restrict__ qkv = args.qkv;
  T* __restrict__ ctx = args.ctx;
  float* __restrict__ lse = args.lse;
  const int s = args.s, heads = args.heads, d = args.d, causal = args.causal;
  const DropArgs drop = args.drop;
  __shared__ __attribute__((aligned(16))) float so[AF_WAVES * 32 * (D + 4)];
  __shared__ float sml[2][AF_WAVES][32];
  const int tid = threadIdx.x, lane = tid % kWave, half = lane >> 5, l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  // x = (batch, head), y = query block, long blocks first (causal)
  const int head = blockIdx.x % heads, bi = blockIdx.x / heads, q0 = (int)(gridDim.y - 1 - blockIdx.y) * 32;
  const int h = heads * d, query = q0 + l32;
  const int64_t ld = 3 * (int64_t)h;
  const T* base = qkv + (int64_t)bi * s * ld + (int64_t)head * d;
  const uint32_t drow = (uint32_t)(((int64_t)bi * heads + head) * s + query);
  floatx4 qf[D / 8], kf[D / 8];
  af_row<T, D, VEC>(qf, base + (int64_t)(query < s ? query : s - 1) * ld, half, d);
  floatx16 o[D / 32];
  af_zero<D>(o);
  float m = -INFINITY, l = 0.f;
  const int end = causal && q0 + 32 < s ? q0 + 32 : s;   // keys
  auto load_k = [&](int k0) {
    const int key = k0 + l32;
    af_row<T, D, VEC>(kf, base + h + (int64_t)(key < s ? key : s - 1) * ld, half, d);
  };
  if (wave * 32 < end) load_k(wave * 32);
  for (int k0 = wave * 32; k0 < end; k0 += AF_WAVES * 32) {
    AfTile<D, D <= 64 ? D / 32 : 1> vt;
    af_ahead<T>(vt, base + 2 * h, ld, k0, s, d, half, l32);
    floatx16 sc = af_dot<D>(kf, qf);
    if (k0 + AF_WAVES * 32 < end) load_k(k0 + AF_WAVES * 32);
    float mx = -INFINITY;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int key = k0 + 8 * (r >> 2) + 4 * half + (r & 3);
      sc[r] = (key >= s || (causal && key > query)) ? -INFINITY : sc[r];
      mx = fmaxf(mx, sc[r]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float m_new = fmaxf(m, mx * scale), alpha = af_exp(m - m_new);
    m = m_new;
    l *= alpha;
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[db][r] *= alpha;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      sc[r] = af_exp(__builtin_fmaf(sc[r], scale, -m));
      l += sc[r];   // the softmax is normalised before the dropout
    }
    if (drop.thr != 0) {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const uint32_t w = drop_row_word(drop, drow, (uint32_t)(k0 + 8 * g + 4 * half) >> 2);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (!drop_keep(drop, w, e)) sc[4 * g + e] = 0.f;
      }
    }
    af_weighted<T>(o, vt, base + 2 * h, ld, k0, s, d, sc, half, l32);
  }
  l += __shfl_xor(l, 32, 64);
  af_put<D>(so, o, wave, half, l32);
  if (half == 0) { sml[0][wave][l32] = m; sml[1][wave][l32] = l; }
  __syncthreads();
  float probe = 0.f;
  const bool whole = d % 4 == 0 && (reinterpret_cast<uintptr_t>(ctx) & (4 * sizeof(T) - 1)) == 0;
  for (int i = tid; i < 32 * D / 4; i += AF_WAVES * kWave) {   // four columns at a time: the weights are a row's
    const int row = i / (D / 4), e = i % (D / 4) * 4;
    if (q0 + row >= s || e >= d) continue;
    float mm = sml[0][0][row];
#pragma unroll
    for (int w = 1; w < AF_WAVES; ++w) mm = fmaxf(mm, sml[0][w][row]);
    floatx4 num = {0.f, 0.f, 0.f, 0.f};
    float den = 0.f;
#pragma unroll
    for (int w = 0; w < AF_WAVES; ++w) {   // a wave without a tile: m = -inf, weight 0
      const float a = af_exp(sml[0][w][row] - mm);
      const floatx4 x = *reinterpret_cast<const floatx4*>(so + (w * 32 + row) * (D + 4) + e);
#pragma unroll
      for (int j = 0; j < 4; ++j) num[j] += a * x[j];
      den += a * sml[1][w][row];
    }
    const float inv = (drop.thr != 0 ? drop.scale : 1.0f) / den;
    typedef T Tx4 __attribute__((ext_vector_type(4)));
    Tx4 out;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (e + j < d) probe = ar_probe(probe, num[j] * inv);
      out[j] = from_f32<T>(num[j] * inv);
    }
    T* to = ctx + ((int64_t)bi * s + q0 + row) * h + (int64_t)head * d + e;
    if (whole) *reinterpret_cast<Tx4*>(to) = out;
    else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (e + j < d) to[j] = out[j];
    }
    if (lse && e == 0) lse[((int64_t)bi * heads + head) * s + q0 + row] = mm + logf(den);
  }
  if (af_any(so + D, probe, wave)) af_rows<T>((int)(gridDim.y - 1 - blockIdx.y), wave, [](const AfArgs<T>& a, int i, int ln, int64_t at3, int64_t at, int64_t stat) {
    ar_fwd<T>(a.qkv + at3, a.ctx + at, a.lse, i, a.s, a.heads * a.d, a.d, a.causal, 1.0f / sqrtf((float)a.d), stat, a.drop, ln);
  });
}

// dQ, and delta = rowsum(dO * O) for the key-side kernel.
template <typename T, int D, bool VEC>
__global__ __launch_bounds__(AF_WAVES* kWave) void attn_f32_bwd_dq_kernel(AfArgs<T> args, float scale) {
  const T* __restrict__ qkv = args.qkv;
  const T* __restrict__ ctx = args.ctx;
  const T* __restrict__ dctx = args.dctx;
  const float* __restrict__ lse = args.lse;
  T* __restrict__ dqkv = args.dqkv;
  float* __restrict__ delta = args.delta;
  const int s = args.s, heads = args.heads, d = args.d, causal = args.causal;
  const DropArgs drop = args.drop;
  __shared__ __attribute__((aligned(16))) float so[AF_WAVES * 32 * (D + 4)];
  const int tid = threadIdx.x, lane = tid % kWave, half = lane >> 5, l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int head = blockIdx.x % heads, bi = blockIdx.x / heads, q0 = (int)(gridDim.y - 1 - blockIdx.y) * 32;
  const int h = heads * d, query = q0 + l32, qrow = query < s ? query : s - 1;
  const int64_t ld = 3 * (int64_t)h, orow = ((int64_t)bi * s + qrow) * h + (int64_t)head * d;
  const T* base = qkv + (int64_t)bi * s * ld + (int64_t)head * d;
  const int64_t sbase = ((int64_t)bi * heads + head) * s;
  floatx4 qf[D / 8], gf[D / 8], rf[D / 8];
  af_row<T, D, VEC>(qf, base + (int64_t)qrow * ld, half, d);
  af_row<T, D, VEC>(gf, dctx + orow, half, d);
  af_row<T, D, VEC>(rf, ctx + orow, half, d);
  float dl = 0.f;
#pragma unroll
  for (int g = 0; g < D / 8; ++g)
#pragma unroll
    for (int i = 0; i < 4; ++i) dl = fmaf(gf[g][i], rf[g][i], dl);
  dl += __shfl_xor(dl, 32, 64);
  if (wave == 0 && half == 0 && query < s) delta[sbase + query] = dl;
  const float l = lse[sbase + qrow];
  floatx16 dq[D / 32];
  af_zero<D>(dq);
  const int end = causal && q0 + 32 < s ? q0 + 32 : s;
  for (int k0 = wave * 32; k0 < end; k0 += AF_WAVES * 32) {
    const int key0 = k0 + l32, krow = key0 < s ? key0 : s - 1;
    af_row<T, D, VEC>(rf, base + h + (int64_t)krow * ld, half, d);
    AfTile<D, D <= 64 || (D == 96 && VEC) ? D / 32 : (D == 96 ? 1 : 2)> kt;
    af_ahead<T>(kt, base + h, ld, k0, s, d, half, l32);
    const floatx16 sc = af_dot<D>(rf, qf);
    af_row<T, D, VEC>(rf, base + 2 * h + (int64_t)krow * ld, half, d);
    floatx16 ds = af_dot<D>(rf, gf);
    if (drop.thr != 0) {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const uint32_t w = drop_row_word(drop, (uint32_t)(sbase + query), (uint32_t)(k0 + 8 * g + 4 * half) >> 2);
#pragma unroll
        for (int e = 0; e < 4; ++e) ds[4 * g + e] = drop_keep(drop, w, e) ? ds[4 * g + e] * drop.scale : 0.f;
      }
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int key = k0 + 8 * (r >> 2) + 4 * half + (r & 3);
      const float p = af_exp(__builtin_fmaf(sc[r], scale, -l));
      ds[r] = (key >= s || (causal && key > query)) ? 0.f : p * (ds[r] - dl);
    }
    af_weighted<T>(dq, kt, base + h, ld, k0, s, d, ds, half, l32);
  }
  af_put<D>(so, dq, wave, half, l32);
  __syncthreads();
  float probe = 0.f;
  for (int i = tid; i < 32 * D; i += AF_WAVES * kWave) {
    const int row = i / D, e = i % D;
    if (q0 + row >= s || e >= d) continue;
    const float v = af_get_sum<D>(so, row, e) * scale;
    probe = ar_probe(probe, v);
    dqkv[((int64_t)bi * s + q0 + row) * ld + (int64_t)head * d + e] = from_f32<T>(v);
  }
  if (af_any(so + D, probe, wave)) af_rows<T>((int)(gridDim.y - 1 - blockIdx.y), wave, [](const AfArgs<T>& a, int i, int ln, int64_t at3, int64_t at, int64_t stat) {
    ar_dq<T>(a.qkv + at3, a.ctx + at, a.dctx + at, a.lse, a.dqkv + at3, i, a.s, a.heads * a.d, a.d, a.causal, 1.0f / sqrtf((float)a.d), stat, a.drop, ln);
  });
}

// dK and dV.
template <typename T, int D, bool VEC>
__global__ __launch_bounds__(AF_WAVES* kWave) void attn_f32_bwd_dkv_kernel(AfArgs<T> args, float scale) {
  const T* __restrict__ qkv = args.qkv;
  const T* __restrict__ dctx = args.dctx;
  const float* __restrict__ lse = args.lse;
  const float* __restrict__ delta = args.delta;
  T* __restrict__ dqkv = args.dqkv;
  const int s = args.s, heads = args.heads, d = args.d, causal = args.causal;
  const DropArgs drop = args.drop;
  __shared__ __attribute__((aligned(16))) float so[AF_WAVES * 32 * (D + 4)];
  const int tid = threadIdx.x, lane = tid % kWave, half = lane >> 5, l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int head = blockIdx.x % heads, bi = blockIdx.x / heads, kb0 = (int)blockIdx.y * 32;   // early keys (most queries) first
  const int h = heads * d, key = kb0 + l32, krow = key < s ? key : s - 1;
  const int64_t ld = 3 * (int64_t)h, sbase = ((int64_t)bi * heads + head) * s;
  const T* base = qkv + (int64_t)bi * s * ld + (int64_t)head * d;
  const T* gbase = dctx + (int64_t)bi * s * h + (int64_t)head * d;
  floatx4 kf[D / 8], vf[D / 8], rf[D / 8];
  af_row<T, D, VEC>(kf, base + h + (int64_t)krow * ld, half, d);
  af_row<T, D, VEC>(vf, base + 2 * h + (int64_t)krow * ld, half, d);
  floatx16 dk[D / 32], dv[D / 32];
  af_zero<D>(dk);
  af_zero<D>(dv);
  for (int q0 = (causal ? kb0 : 0) + wave * 32; q0 < s; q0 += AF_WAVES * 32) {
    const int qr = q0 + l32, qrow = qr < s ? qr : s - 1;
    af_row<T, D, VEC>(rf, base + (int64_t)qrow * ld, half, d);
    AfTile<D, D <= 64 ? D / 32 : (D == 96 ? 1 : 2)> gt, qt;
    af_ahead<T>(gt, gbase, h, q0, s, d, half, l32);
    af_ahead<T>(qt, base, ld, q0, s, d, half, l32);
    const floatx16 sc = af_dot<D>(rf, kf);
    af_row<T, D, VEC>(rf, gbase + (int64_t)qrow * h, half, d);
    const floatx16 dp = af_dot<D>(rf, vf);
    floatx16 pr, ds;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int q = q0 + 8 * (r >> 2) + 4 * half + (r & 3);
      const bool in = q < s && !(causal && q < key);
      const int64_t at = sbase + (q < s ? q : s - 1);
      const float e = af_exp(__builtin_fmaf(sc[r], scale, -lse[at]));
      const float p = in ? e : 0.f;
      float f = 1.0f;
      if (drop.thr != 0 && in)
        f = drop_keep(drop, drop_row_word(drop, (uint32_t)(sbase + q), (uint32_t)key >> 2), key & 3) ? drop.scale : 0.f;
      pr[r] = p * f;
      ds[r] = in ? p * (dp[r] * f - delta[at]) : 0.f;
    }
    af_weighted<T>(dv, gt, gbase, h, q0, s, d, pr, half, l32);
    af_weighted<T>(dk, qt, base, ld, q0, s, d, ds, half, l32);
  }
  af_put<D>(so, dk, wave, half, l32);
  __syncthreads();
  float probe = 0.f;
  for (int i = tid; i < 32 * D; i += AF_WAVES * kWave) {
    const int row = i / D, e = i % D;
    if (kb0 + row >= s || e >= d) continue;
    const float v = af_get_sum<D>(so, row, e) * scale;
    probe = ar_probe(probe, v);
    dqkv[((int64_t)bi * s + kb0 + row) * ld + h + (int64_t)head * d + e] = from_f32<T>(v);
  }
  __syncthreads();
  af_put<D>(so, dv, wave, half, l32);
  __syncthreads();
  for (int i = tid; i < 32 * D; i += AF_WAVES * kWave) {
    const int row = i / D, e = i % D;
    if (kb0 + row >= s || e >= d) continue;
    const float v = af_get_sum<D>(so, row, e);
    probe = ar_probe(probe, v);
    dqkv[((int64_t)bi * s + kb0 + row) * ld + 2 * h + (int64_t)head * d + e] = from_f32<T>(v);
  }
  if (af_any(so + D, probe, wave)) af_rows<T>((int)blockIdx.y, wave, [](const AfArgs<T>& a, int i, int ln, int64_t at3, int64_t at, int64_t stat) {
    ar_dkv<T>(a.qkv + at3, a.dctx + at, a.lse, a.delta, a.dqkv + at3, i, a.s, a.heads * a.d, a.d, a.causal, 1.0f / sqrtf((float)a.d), stat, a.drop, ln);
  });
}

template <typename T, int D, bool VEC>
inline hipError_t af_fwd(const T* qkv, T* ctx, float* lse, int b, int s, int heads, int d, int causal, const DropArgs& drop, hipStream_t st) {
  const dim3 grid((unsigned)(heads * b), (unsigned)((s + 31) / 32));
  const AfArgs<T> a{qkv, ctx, lse, nullptr, nullptr, nullptr, s, heads, d, causal, drop};
  hipLaunchKernelGGL((attn_f32_fwd_kernel<T, D, VEC>), grid, dim3(AF_WAVES * kWave), 0, st, a, 1.0f / sqrtf((float)d));
  return hipGetLastError();
}
template <typename T, int D, bool VEC>
inline hipError_t af_bwd(const T* qkv, const T* ctx, const float* lse, const T* dctx, T* dqkv, float* delta, int b, int s, int heads, int d,
                         int causal, const DropArgs& drop, hipStream_t st) {
  const dim3 grid((unsigned)(heads * b), (unsigned)((s + 31) / 32)), block(AF_WAVES * kWave);
  const float scale = 1.0f / sqrtf((float)d);
  const AfArgs<T> a{qkv, const_cast<T*>(ctx), const_cast<float*>(lse), dctx, dqkv, delta, s, heads, d, causal, drop};
  hipLaunchKernelGGL((attn_f32_bwd_dq_kernel<T, D, VEC>), grid, block, 0, st, a, scale);
  hipLaunchKernelGGL((attn_f32_bwd_dkv_kernel<T, D, VEC>), grid, block, 0, st, a, scale);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_attention_fwd_f32(const T* qkv, T* ctx, float* lse, int b, int s, int heads, int d, int causal, const DropArgs& drop, hipStream_t st) {
  const bool vec = attn_f32_vec<T>(qkv, qkv, qkv, d);
#define VARUNA_AF(D_) \
  if (d <= D_) return vec ? af_fwd<T, D_, true>(qkv, ctx, lse, b, s, heads, d, causal, drop, st) : af_fwd<T, D_, false>(qkv, ctx, lse, b, s, heads, d, causal, drop, st);
  VARUNA_AF(32) VARUNA_AF(64) VARUNA_AF(96) VARUNA_AF(128)
#undef VARUNA_AF
  return hipErrorInvalidConfiguration;
}
template <typename T>
hipError_t launch_attention_bwd_f32(const T* qkv, const T* ctx, const float* lse, const T* dctx, T* dqkv, float* delta, int b, int s,
                                    int heads, int d, int causal, const DropArgs& drop, hipStream_t st) {
  const bool vec = attn_f32_vec<T>(qkv, ctx, dctx, d);
#define VARUNA_AF(D_) \
  if (d <= D_) return vec ? af_bwd<T, D_, true>(qkv, ctx, lse, dctx, dqkv, delta, b, s, heads, d, causal, drop, st) \
                          : af_bwd<T, D_, false>(qkv, ctx, lse, dctx, dqkv, delta, b, s, heads, d, causal, drop, st);
  VARUNA_AF(32) VARUNA_AF(64) VARUNA_AF(96) VARUNA_AF(128)
#undef VARUNA_AF
  return hipErrorInvalidConfiguration;
}

}  // namespace varuna
