// fp32 attention on the matrix cores in tiles of 16 (v_mfma_f32_16x16x4_f32), head dims up to 128 that are multiples of 4 (padded to D in {32, 64, 96, 128}
// with zeros), any sequence length: what attention_f32.h does in tiles of 32.  The rate of the products is the same.
//
// What bounds it: the chain of one wave (its loads, its products at 32 clocks each, the exchange at the end) and, on many rows, the fp32 matrix
// rate.  A 16x16 tile takes a quarter of a 32x32 tile's products and there are four times as many for the waves to share; all loads of a tile are on
// their way before its first product; the backward is one launch, whose key side sums delta itself.  Which form a call takes, with both
// sides measured: attn_f32_16 in attention.h.
//
// A workgroup of 4 waves has 16 queries (forward, dQ) or 16 keys (dK, dV) of one head; its waves take every fourth 16 rows of the other side
// and meet in LDS at the end, in a fixed order.  Scores lie in the result with the softmax row as column: lane L holds rows 4*(L/16) + r (r = 0..3)
// of column L%16, which is the second product's operand as it stands.  A score adds its terms in the order of the other forms (k-values 8g + i,
// then 8g + 4 + i: attention_rows.h) and is theirs to the bit.
#pragma once
#include "attention_f32.h"

namespace varuna {

constexpr int AW_WAVES = 4;

// One row of d columns, four of every 16 in each of the row's four lanes: columns 16G + 4*quad .. +3.
template <int D>
struct AwRow {
  floatx4 x[D / 16];
  __device__ __forceinline__ void load(const float* __restrict__ row, int quad, int d) {
#pragma unroll
    for (int g = 0; g < D / 16; ++g) {
      const int e = 16 * g + 4 * quad;
      x[g] = *reinterpret_cast<const floatx4*>(row + (e < d ? e : 0));
      if (e >= d) x[g] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
  }
  // As score operands: of 8 columns 8g .. 8g + 7, which quads 0 and 1 hold (even g) or quads 2 and 3, one product takes 8g + 0, 4, 1, 5 in quads
  // 0 .. 3 and the next one 8g + 2, 6, 3, 7.  One exchange between the half waves gives an operand of both groups.
  __device__ __forceinline__ void spread() {
#pragma unroll
    for (int g = 0; g < D / 16; ++g)
#pragma unroll
      for (int w = 0; w < 2; ++w) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x[g][2 * w]), __float_as_uint(x[g][2 * w + 1]), false, false);
        x[g][2 * w] = __uint_as_float(r[0]);       // of columns 16g .. 16g + 7
        x[g][2 * w + 1] = __uint_as_float(r[1]);   // of columns 16g + 8 .. 16g + 15
      }
  }
};
// acc[row of a][row of b] over the head dim, of spread rows
template <int D>
__device__ __forceinline__ floatx4 aw_dot(const AwRow<D>& a, const AwRow<D>& b) {
  floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int g = 0; g < D / 8; ++g)
#pragma unroll
    for (int w = 0; w < 2; ++w)
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x[g / 2][2 * w + (g & 1)], b.x[g / 2][2 * w + (g & 1)], acc, 0, 0, 0);
  return acc;
}
// The tile's rows 4*quad + r, columns 16*db + lane%16 (rows past the end repeat the last one: their weight is zero; columns past the end reach
// only results that are not stored).
template <int D>
struct AwCols {
  float x[D / 16][4];
  __device__ __forceinline__ void load(const float* __restrict__ base, int64_t ld, int row0, int rows, int quad, int i16, int d) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = row0 + 4 * quad + r;
      const float* p = base + (int64_t)(row < rows ? row : rows - 1) * ld;
#pragma unroll
      for (int db = 0; db < D / 16; ++db) x[db][r] = p[16 * db + i16 < d ? 16 * db + i16 : 0];
    }
  }
};
// acc[db][column of the tile][column of the weights] += sum over the tile's rows
template <int D>
__device__ __forceinline__ void aw_weighted(floatx4 (&acc)[D / 16], const AwCols<D>& t, const floatx4& w) {
#pragma unroll
  for (int db = 0; db < D / 16; ++db)
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[db] = __builtin_amdgcn_mfma_f32_16x16x4f32(t.x[db][r], w[r], acc[db], 0, 0, 0);
}
// Partial results in LDS, [wave][column][D + 4]: acc[db][r] is element 16*db + 4*quad + r of column lane%16.
template <int D>
__device__ __forceinline__ void aw_put(float* sm, const floatx4 (&acc)[D / 16], int wave, int quad, int i16) {
#pragma unroll
  for (int db = 0; db < D / 16; ++db) *reinterpret_cast<floatx4*>(sm + (wave * 16 + i16) * (D + 4) + 16 * db + 4 * quad) = acc[db];
}
template <int D>
__device__ __forceinline__ floatx4 aw_sum(const float* sm, int row, int e) {
  floatx4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int w = 0; w < AW_WAVES; ++w) v += *reinterpret_cast<const floatx4*>(sm + (w * 16 + row) * (D + 4) + e);
  return v;
}
__device__ __forceinline__ float aw_probe(float t, const floatx4& v) {
#pragma unroll
  for (int j = 0; j < 4; ++j) t = ar_probe(t, v[j]);
  return t;
}
// Whether any thread of the block saw a result that is not finite.
__device__ __forceinline__ bool aw_any(float* flags, float probe, int wave, int lane) {
  const float mine = __ballot(!(probe == 0.f)) != 0 ? 1.f : 0.f;
  if (lane == 0) flags[wave] = mine;
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(flags[0] + flags[1] + flags[2] + flags[3] != 0.f);
}

struct AwArgs {
  const float* qkv; float* ctx; float* lse;
  const float* dctx; float* dqkv; float* delta;
  int s, heads, d, causal;
  DropArgs drop;
};

template <int D>
__global__ __launch_bounds__(AW_WAVES* kWave) void attn_f32_16_fwd_kernel(AwArgs a, float scale) {
  __shared__ __attribute__((aligned(16))) float so[AW_WAVES * 16 * (D + 4)];
  __shared__ float sml[2][AW_WAVES][16], flags[AW_WAVES];
  const int tid = threadIdx.x, lane = tid % kWave, quad = lane >> 4, i16 = lane & 15, s = a.s, d = a.d;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int head = blockIdx.x % a.heads, bi = blockIdx.x / a.heads, q0 = (int)(gridDim.y - 1 - blockIdx.y) * 16;
  const int h = a.heads * d, query = q0 + i16;
  const int64_t ld = 3 * (int64_t)h, tok = (int64_t)bi * s, stat = ((int64_t)bi * a.heads + head) * s;
  const float* base = a.qkv + tok * ld + head * d;
  AwRow<D> qf, kf;
  AwCols<D> vt;
  qf.load(base + (int64_t)(query < s ? query : s - 1) * ld, quad, d);
  floatx4 o[D / 16];
#pragma unroll
  for (int db = 0; db < D / 16; ++db) o[db] = floatx4{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.f;
  const int end = a.causal && q0 + 16 < s ? q0 + 16 : s;   // keys
  for (int k0 = wave * 16; k0 < end; k0 += AW_WAVES * 16) {
    kf.load(base + h + (int64_t)(k0 + i16 < s ? k0 + i16 : s - 1) * ld, quad, d);
    vt.load(base + 2 * h, ld, k0, s, quad, i16, d);
    __builtin_amdgcn_sched_barrier(0);   // both are on their way before the first wait
    if (k0 == wave * 16) qf.spread();
    kf.spread();
    floatx4 sc = aw_dot<D>(kf, qf);
    float mx = -INFINITY;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int key = k0 + 4 * quad + r;
      sc[r] = (key >= s || (a.causal && key > query)) ? -INFINITY : sc[r];
      mx = fmaxf(mx, sc[r]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16, kWave));
    mx = fmaxf(mx, __shfl_xor(mx, 32, kWave));
    // (a tile past the causal diagonal of a query is all -inf: the reference stays, and so do the sums)
    const float m_new = fmaxf(m, mx * scale), ref = m_new == -INFINITY ? 0.f : m_new, alpha = af_exp(m - ref);
    m = m_new;
    l *= alpha;
#pragma unroll
    for (int db = 0; db < D / 16; ++db) o[db] *= alpha;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      sc[r] = af_exp(__builtin_fmaf(sc[r], scale, -ref));
      l += sc[r];   // the softmax is normalised before the dropout
    }
    if (a.drop.thr != 0) {
      const uint32_t w = drop_row_word(a.drop, (uint32_t)(stat + query), (uint32_t)(k0 + 4 * quad) >> 2);
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (!drop_keep(a.drop, w, r)) sc[r] = 0.f;
    }
    aw_weighted<D>(o, vt, sc);
  }
  l += __shfl_xor(l, 16, kWave);
  l += __shfl_xor(l, 32, kWave);
  aw_put<D>(so, o, wave, quad, i16);
  if (quad == 0) { sml[0][wave][i16] = m; sml[1][wave][i16] = l; }
  __syncthreads();
  float probe = 0.f;
  for (int i = tid; i < 16 * D / 4; i += AW_WAVES * kWave) {   // four columns at a time: the weights are a row's
    const int row = i / (D / 4), e = i % (D / 4) * 4;
    if (q0 + row >= s || e >= d) continue;
    float mm = sml[0][0][row];
#pragma unroll
    for (int w = 1; w < AW_WAVES; ++w) mm = fmaxf(mm, sml[0][w][row]);
    floatx4 num = {0.f, 0.f, 0.f, 0.f};
    float den = 0.f;
#pragma unroll
    for (int w = 0; w < AW_WAVES; ++w) {   // a wave without a tile: m = -inf, weight 0
      const float f = af_exp(sml[0][w][row] - mm);
      num += f * *reinterpret_cast<const floatx4*>(so + (w * 16 + row) * (D + 4) + e);
      den += f * sml[1][w][row];
    }
    num *= (a.drop.thr != 0 ? a.drop.scale : 1.0f) / den;
    probe = aw_probe(probe, num);
    *reinterpret_cast<floatx4*>(a.ctx + (tok + q0 + row) * h + head * d + e) = num;
    if (a.lse && e == 0) a.lse[stat + q0 + row] = mm + logf(den);
  }
  if (aw_any(flags, probe, wave, lane))   // a masked token's infinity or NaN is kept out of the rows that must not see it
    for (int row = q0 + wave; row < q0 + 16 && row < s; row += AW_WAVES)
      ar_fwd<float>(base, a.ctx + tok * h + head * d, a.lse, row, s, h, d, a.causal, scale, stat, a.drop, lane);
}

// dQ and delta: workgroups from the grid's second half; dK and dV: the first half (the longer ones).
template <int D>
__global__ __launch_bounds__(AW_WAVES* kWave) void attn_f32_16_bwd_kernel(AwArgs a, float scale) {
  __shared__ __attribute__((aligned(16))) float so[2][AW_WAVES * 16 * (D + 4)];
  __shared__ float flags[AW_WAVES];
  const int tid = threadIdx.x, lane = tid % kWave, quad = lane >> 4, i16 = lane & 15, s = a.s, d = a.d;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int blocks = (s + 15) / 16;
  const bool keys = (int)blockIdx.y < blocks;
  const int head = blockIdx.x % a.heads, bi = blockIdx.x / a.heads;
  const int r0 = (keys ? (int)blockIdx.y : 2 * blocks - 1 - (int)blockIdx.y) * 16;   // its first key or query, long ones first
  const int h = a.heads * d, own = r0 + i16, orow = own < s ? own : s - 1;
  const int64_t ld = 3 * (int64_t)h, tok = (int64_t)bi * s, stat = ((int64_t)bi * a.heads + head) * s;
  const float* base = a.qkv + tok * ld + head * d;
  const float* gbase = a.dctx + tok * h + head * d;
  const float* cbase = a.ctx + tok * h + head * d;
  // delta of the row that two loaded rows of dO and O belong to, in every lane of its column
  auto row_delta = [&](const AwRow<D>& g, const AwRow<D>& c) {
    float t = 0.f;
#pragma unroll
    for (int k = 0; k < D / 16; ++k)
#pragma unroll
      for (int w = 0; w < 4; ++w) t = fmaf(g.x[k][w], c.x[k][w], t);
    t += __shfl_xor(t, 16, kWave);
    return t + __shfl_xor(t, 32, kWave);
  };
  floatx4 acc[2][D / 16];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int db = 0; db < D / 16; ++db) acc[i][db] = floatx4{0.f, 0.f, 0.f, 0.f};
  AwRow<D> xf, yf;   // of the own rows: Q and dO, or K and V
  float probe = 0.f;
  if (!keys) {
    AwRow<D> cf;
    xf.load(base + (int64_t)orow * ld, quad, d);
    yf.load(gbase + (int64_t)orow * h, quad, d);
    cf.load(cbase + (int64_t)orow * h, quad, d);
    const float l = a.lse[stat + orow];
    const int end = a.causal && r0 + 16 < s ? r0 + 16 : s;
    AwRow<D> kf, vf;
    AwCols<D> kt;
    auto load = [&](int k0) {
      const int64_t at = (int64_t)(k0 + i16 < s ? k0 + i16 : s - 1) * ld;
      kf.load(base + h + at, quad, d);
      vf.load(base + 2 * h + at, quad, d);
      kt.load(base + h, ld, k0, s, quad, i16, d);
      __builtin_amdgcn_sched_barrier(0);
    };
    if (wave * 16 < end) load(wave * 16);
    const float dl = row_delta(yf, cf);
    xf.spread();
    yf.spread();
    if (wave == 0 && quad == 0 && own < s) a.delta[stat + own] = dl;
    for (int k0 = wave * 16; k0 < end; k0 += AW_WAVES * 16) {
      if (k0 != wave * 16) load(k0);
      kf.spread();
      vf.spread();
      const floatx4 sc = aw_dot<D>(kf, xf);
      floatx4 ds = aw_dot<D>(vf, yf);
      if (a.drop.thr != 0) {
        const uint32_t w = drop_row_word(a.drop, (uint32_t)(stat + own), (uint32_t)(k0 + 4 * quad) >> 2);
#pragma unroll
        for (int r = 0; r < 4; ++r) ds[r] = drop_keep(a.drop, w, r) ? ds[r] * a.drop.scale : 0.f;
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int key = k0 + 4 * quad + r;
        const float p = af_exp(__builtin_fmaf(sc[r], scale, -l));
        ds[r] = (key >= s || (a.causal && key > own)) ? 0.f : p * (ds[r] - dl);
      }
      aw_weighted<D>(acc[0], kt, ds);
    }
    aw_put<D>(so[0], acc[0], wave, quad, i16);
    __syncthreads();
    for (int i = tid; i < 16 * D / 4; i += AW_WAVES * kWave) {
      const int row = i / (D / 4), e = i % (D / 4) * 4;
      if (r0 + row >= s || e >= d) continue;
      const floatx4 v = aw_sum<D>(so[0], row, e) * scale;
      probe = aw_probe(probe, v);
      *reinterpret_cast<floatx4*>(a.dqkv + (tok + r0 + row) * ld + head * d + e) = v;
    }
  } else {
    xf.load(base + h + (int64_t)orow * ld, quad, d);
    yf.load(base + 2 * h + (int64_t)orow * ld, quad, d);
    bool first = true;
    for (int q0 = (a.causal ? r0 : 0) + wave * 16; q0 < s; q0 += AW_WAVES * 16) {
      const int64_t q = q0 + i16 < s ? q0 + i16 : s - 1;
      AwRow<D> qf, gf, cf;
      AwCols<D> qt, gt;
      float ls[4];
      qf.load(base + q * ld, quad, d);
      gf.load(gbase + q * h, quad, d);
      cf.load(cbase + q * h, quad, d);
      qt.load(base, ld, q0, s, quad, i16, d);
      gt.load(gbase, h, q0, s, quad, i16, d);
#pragma unroll
      for (int r = 0; r < 4; ++r) ls[r] = a.lse[stat + (q0 + 4 * quad + r < s ? q0 + 4 * quad + r : s - 1)];
      __builtin_amdgcn_sched_barrier(0);
      const float dl = row_delta(gf, cf);   // of query q0 + lane % 16
      if (first) { xf.spread(); yf.spread(); first = false; }
      qf.spread();
      gf.spread();
      const floatx4 sc = aw_dot<D>(qf, xf);
      const floatx4 dp = aw_dot<D>(gf, yf);
      floatx4 pr, ds;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int qr = q0 + 4 * quad + r;
        const bool in = qr < s && !(a.causal && qr < own);
        const float e = af_exp(__builtin_fmaf(sc[r], scale, -ls[r])), p = in ? e : 0.f;
        float f = 1.0f;
        if (a.drop.thr != 0 && in) f = drop_keep(a.drop, drop_row_word(a.drop, (uint32_t)(stat + qr), (uint32_t)own >> 2), own & 3) ? a.drop.scale : 0.f;
        pr[r] = p * f;
        const float dlr = __shfl(dl, 4 * quad + r, kWave);
        ds[r] = in ? p * (dp[r] * f - dlr) : 0.f;
      }
      aw_weighted<D>(acc[0], qt, ds);
      aw_weighted<D>(acc[1], gt, pr);
    }
    aw_put<D>(so[0], acc[0], wave, quad, i16);
    aw_put<D>(so[1], acc[1], wave, quad, i16);
    __syncthreads();
    for (int i = tid; i < 16 * D / 4; i += AW_WAVES * kWave) {
      const int row = i / (D / 4), e = i % (D / 4) * 4;
      if (r0 + row >= s || e >= d) continue;
      const floatx4 dk = aw_sum<D>(so[0], row, e) * scale, dv = aw_sum<D>(so[1], row, e);
      probe = aw_probe(aw_probe(probe, dk), dv);
      float* to = a.dqkv + (tok + r0 + row) * ld + h + head * d + e;
      *reinterpret_cast<floatx4*>(to) = dk;
      *reinterpret_cast<floatx4*>(to + h) = dv;
    }
  }
  if (!aw_any(flags, probe, wave, lane)) return;
  for (int row = r0 + wave; row < r0 + 16 && row < s; row += AW_WAVES) {
    if (keys) ar_dkv<float>(base, gbase, a.lse, a.delta, a.dqkv + tok * ld + head * d, row, s, h, d, a.causal, scale, stat, a.drop, lane, cbase);
    else ar_dq<float>(base, cbase, gbase, a.lse, a.dqkv + tok * ld + head * d, row, s, h, d, a.causal, scale, stat, a.drop, lane);
  }
}

}  // namespace varuna
