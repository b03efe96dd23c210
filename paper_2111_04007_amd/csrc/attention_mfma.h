// bf16 MFMA flash-style attention for gfx950: forward, and a two-kernel
// deterministic backward (no atomics).  Head dim D in {64, 96, 128}, sequence
// length a multiple of 128; with EDGE any sequence length and any head dim d that
// is a multiple of 8, in the next D of {32, 64, 96, 128}.  qkv is [b*s, 3h] (Q | K | V column blocks, head j at
// column j*D of each), ctx / dctx are [b*s, h], lse / delta are [b, heads, s] fp32.
//
// The EDGE form works out rows that are not finite again one by one (attention_rows.h), so that an infinity or NaN of a
// masked token does not reach them.
//
// All three kernels keep tiles of two matrices in LDS (64 rows each; dK/dV 32, twice)
// and hold the other operands in registers.  Products use
// v_mfma_f32_32x32x16_bf16 whose operand layout is: row operand lane L -> row
// L%32, k = 8*(L/32)..+7; column operand likewise; result lane L -> column L%32,
// rows 8*(r/4) + 4*(L/32) + r%4 for the 16 registers r.  Scores are computed
// "transposed" (tile rows as the MFMA row operand) so that a lane ends up with 16
// scores of ONE softmax row per 32x32 block: row statistics need one cross-half
// shuffle, and the probabilities are already laid out as the column operand of
// the following product, whose other operand comes out of LDS through the
// transposing read ds_read_b64_tr_b16 (the k-slot order of the two operands
// then agrees by construction).
//
//   forward (per 128-query workgroup, 32 queries per wave; K, V tiles in LDS):
//     S^T = K Q^T ; online softmax in base 2 ; O^T += V^T P^T
//   backward dQ (same geometry): S^T, dP^T = V dO^T ; dS = P (dP - delta) ;
//     dQ^T += K^T dS^T ; also writes delta = rowsum(dO * O)
//   backward dK/dV (per 128-key workgroup, 32 keys per wave; Q, dO tiles in LDS):
//     S = Q K^T, dP = dO V^T ; dV^T += dO^T P ; dK^T += Q^T dS
//
// What bounds them: a wave's chain of fragment reads, products, softmax arithmetic and tile exchange.  The products alone, with the
// same barriers, take a third to a half of a kernel's time, and two waves of a SIMD overlap only in part; so what pays is what
// shortens a wave's chain or keeps two waves on a SIMD: no bank conflicts (a fifth of the LDS cycles before), tile loads that
// need neither 64-bit addresses nor masks (buffer loads), nothing in the loop that waits for the next tile's loads (a
// register spill does), the mask's arithmetic on the diagonal only.
#pragma once
#include "attention_rows.h"
#include "common.h"

namespace varuna {

typedef short at_shortx4 __attribute__((ext_vector_type(4)));

template <int D>
struct AttnCfg {
  static_assert(D == 32 || D == 64 || D == 96 || D == 128, "head dim");
  // LDS row pitch in elements: an odd multiple of 64 bytes, so that four consecutive rows' 64-byte pieces, which 32 lanes of a
  // transposing read take at once, lie in different quarters of the 256 bytes of banks.  Within such a piece the 16-byte chunks
  // of row r are XOR-permuted by (r / 4) % 4: 16 consecutive rows of a 16-byte read fall into different banks as well.
  static constexpr int PITCH = D == 32 ? 32 : (D == 128 ? 160 : 96);
  static constexpr int CH = D / 8;             // 16-byte chunks per row
  static constexpr int KD = D / 16;            // k-steps over the head dim
  static constexpr int DB = D / 32;            // 32-wide blocks of the head dim
};

// Rows of the same ROWS tokens (or of ROWS tokens each) of two matrices, D columns, on their way to LDS: waves 0 and 1 of the
// workgroup's four move the first, 2 and 3 the second.  Buffer loads: what lies past the end of a sequence (EDGE) is outside
// the buffer and reads as zero, and so are a head's missing columns, whose lanes hold an offset outside.
template <int D, bool EDGE, int ROWS>
struct AttnTilePair {
  static constexpr int CH = AttnCfg<D>::CH, CPT = ROWS * CH / 128;   // chunks per row, per thread
  static constexpr bool WHOLE = CH == 8 || CH == 16;                 // a load takes whole rows (else 64-byte quarters)
  static constexpr int NV = WHOLE ? 1 : CH / 4;
  static constexpr uint32_t OUTSIDE = 0xfffffff0u;   // past any row of the tile (a row has up to 48 MB)
  floatx4 v[CPT];
  uint32_t voff[NV];
  int64_t ld2;         // bytes per row
  const char* base;    // the sequence's first row
  int at;
  __device__ __forceinline__ void init(const bf16* first_row, int64_t row_stride, int t, int cols) {
    base = reinterpret_cast<const char*>(first_row);
    ld2 = row_stride * 2;
    const int r = WHOLE ? t / CH : t / 4, c = WHOLE ? t % CH : t % 4;
#pragma unroll
    for (int i = 0; i < NV; ++i) voff[i] = EDGE && (c + 4 * i) * 8 >= cols ? OUTSIDE : (uint32_t)(r * ld2 + (c + 4 * i) * 16);
    at = (r * AttnCfg<D>::PITCH + (c & ~3) * 8 + ((c ^ (r >> 2)) & 3) * 8) * 2;
  }
  // piece i: its row (beyond the thread's first) and its place in the row (bytes beyond the thread's first)
  static __device__ __forceinline__ constexpr int row_of(int i) { return WHOLE ? i * (128 / CH) : i / (CH / 4) * 32; }
  __device__ __forceinline__ void load(int row0, int rows, int cols) {
#if defined(__HIP_DEVICE_COMPILE__)  // the buffer builtins exist in the device pass only
    const int left = rows - row0;
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(base + row0 * ld2), 0,
                                                        EDGE ? (uint32_t)(((left < ROWS ? left : ROWS) - 1) * ld2 + cols * 2) : OUTSIDE, 0x00020000);
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
      const uint32_t rows_on = (uint32_t)(row_of(i) * ld2);   // (EDGE: part of the offset that the range check sees)
      const uint32_t off = EDGE ? __builtin_elementwise_add_sat(voff[WHOLE ? 0 : i % NV], rows_on) : voff[WHOLE ? 0 : i % NV];
      v[i] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)off, EDGE ? 0 : (int)rows_on, 0));
    }
#endif
  }
  __device__ __forceinline__ void store(bf16* lds) const {
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
      const int flip = (row_of(i) >> 2 & 3) * 16;   // the swizzle of the piece's row against that of the thread's first
      *reinterpret_cast<floatx4*>(reinterpret_cast<char*>(lds) + (at ^ flip) + row_of(i) * AttnCfg<D>::PITCH * 2 + (WHOLE ? 0 : i % NV * 64)) = v[i];
    }
  }
};

// Columns 16t + 8*(lane/32) .. +7 of one row of `cols` columns for every k-step t; zero past the end of the row.
template <int D, bool EDGE>
__device__ __forceinline__ void at_load_row(bf16x8 (&f)[AttnCfg<D>::KD], const bf16* __restrict__ row, int hf, int cols) {
#pragma unroll
  for (int t = 0; t < AttnCfg<D>::KD; ++t) {
    const int c = 16 * t + 8 * hf;
    if (EDGE && c >= cols) f[t] = bf16x8{};
    else f[t] = *reinterpret_cast<const bf16x8*>(row + c);
  }
}

// Row operand from an LDS tile: row (row_base + lane%32), columns 16t + 8*(lane/32) .. +7.  row_base: a multiple of 32.
template <int D>
__device__ __forceinline__ bf16x8 at_row_frag(const bf16* tile, int row_base, int t, int lane) {
  const int c = ((t & 1) * 2 + (lane >> 5)) ^ (lane >> 2 & 3);
  return *reinterpret_cast<const bf16x8*>(tile + (row_base + (lane & 31)) * AttnCfg<D>::PITCH + (t >> 1) * 32 + c * 8);
}

// Transposed row operand: operand row = tile column (col_base + lane%32); its 8 k-slots are
// tile rows r0 + 4*(lane/32) + {0..3} and r0 + 8 + 4*(lane/32) + {0..3} -- the order in
// which a lane holds the rows of a 32x32 MFMA result, i.e. of P / dS.  r0: a multiple of 16.
template <int D>
__device__ __forceinline__ bf16x8 at_tr_frag(const bf16* tile, int r0, int col_base, int lane) {
  const int j = lane & 15, hf = lane >> 5, c = (lane >> 4 & 1) * 2 + (j >> 1 & 1);
  const bf16* p = tile + (r0 + 4 * hf + (j >> 2)) * AttnCfg<D>::PITCH + col_base + 4 * (j & 1);
  at_shortx4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) at_shortx4*)(p + (c ^ hf) * 8));
  at_shortx4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) at_shortx4*)(p + 8 * AttnCfg<D>::PITCH + (c ^ hf ^ 2) * 8));
  union { struct { at_shortx4 a, b; } s; bf16x8 v; } u;
  u.s.a = lo; u.s.b = hi;
  return u.v;
}

// acc += A B with the accumulator pinned to the accumulation registers.  With one wave per
// SIMD a kernel spreads over both halves of the register file, and left to itself the
// compiler may keep long-lived accumulators in the ordinary half and copy all 16
// registers across around every product.  (No kernel calls it now: the dK/dV kernel did until it fitted two waves per SIMD, where the compiler's own products
// are as fast.  A test holds the wait states.)  The product is opaque to the compiler here, so the
// wait states around it are inserted by hand: two between an operand's last VALU write and the product (a conversion or
// register move may stand directly before it; the product then multiplied what the register held before, now and then:
// dK of d = 32 with dropout up to infinity), and those a later read of the result needs (at_mfma_settle).
__device__ __forceinline__ void at_mfma_acc(floatx16& acc, const bf16x8& a, const bf16x8& b) {
  asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}
__device__ __forceinline__ void at_mfma_settle() { asm volatile("s_nop 15\n\ts_nop 15" ::: "memory"); }

// Value of lane (4*(lane/4) + j) of the same lane quad, j known at compile time after
// unrolling (a DPP quad permutation: no LDS, no wait).
__device__ __forceinline__ uint32_t at_quad_bcast(uint32_t v, int j) {
  switch (j & 3) {
    case 0: return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x00, 0xf, 0xf, false);
    case 1: return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x55, 0xf, 0xf, false);
    case 2: return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xaa, 0xf, 0xf, false);
    default: return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xff, 0xf, 0xf, false);
  }
}

// Dropout mask words for a lane that owns ONE mask row (its query) and, per 32-key block, the
// four 4-key groups g = 0..3 of that row.  The four lanes of a quad own the four rows of the
// same 4x4 mask patches, so each lane generates only the patch of group g = lane%4 and the
// quad exchanges words: out[g] = word (lane%4) of the patch generated by quad lane g.
// row_patch must be the same in all four lanes; col_patch0 is group 0's patch column, group g
// lies two patch columns further per step.
__device__ __forceinline__ void at_drop_row_words(const DropArgs& drop, uint32_t row_patch, uint32_t col_patch0, int lane,
                                                  uint32_t out[4]) {
  const int ql = lane & 3;
  uint32_t own[4];
  drop_patch(drop, row_patch, col_patch0 + 2u * (uint32_t)ql, own);
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const uint32_t t0 = at_quad_bcast(own[0], g), t1 = at_quad_bcast(own[1], g);
    const uint32_t t2 = at_quad_bcast(own[2], g), t3 = at_quad_bcast(own[3], g);
    out[g] = ql == 0 ? t0 : (ql == 1 ? t1 : (ql == 2 ? t2 : t3));
  }
}

// The same words without the quad exchange, for sequence lengths that are no multiple of 4 (the four lanes of a quad
// then straddle two rows of patches).
__device__ __forceinline__ void at_drop_row_words_any(const DropArgs& drop, uint32_t row, uint32_t col_patch0, uint32_t out[4]) {
#pragma unroll
  for (int g = 0; g < 4; ++g) out[g] = drop_row_word(drop, row, col_patch0 + 2u * (uint32_t)g);
}

__device__ __forceinline__ bf16x8 at_pack8(const float* p) {
  bf16x8 r;
#pragma unroll
  for (int i = 0; i < 8; ++i) r[i] = (bf16)p[i];
  return r;
}

// What the rounding in at_pack8 left over.  The EDGE kernels multiply probabilities and score gradients in two parts, p =
// bf16(p) + bf16(p - bf16(p)), which keeps 16 bits of mantissa: the shapes they serve had fp32 factors there (error
// of a bf16 result against 64 bits unchanged: 2.1e-3 forward, 2.4e-3 backward, both the rounding of the output).
__device__ __forceinline__ bf16x8 at_pack8_rest(const float* p, const bf16x8& hi) {
  bf16x8 r;
#pragma unroll
  for (int i = 0; i < 8; ++i) r[i] = (bf16)(p[i] - (float)hi[i]);
  return r;
}

// f(row, lane, head, sequence) for the marked rows of the wave's 32, by the whole wave (attention_rows.h).  What f needs is derived
// anew: values of the kernel's start kept for this rare path would cost its loop registers.
template <typename F>
__device__ __forceinline__ void at_bad_rows(uint32_t bad, int first, int rows, int heads, F&& f) {
  bad = __builtin_amdgcn_readfirstlane(bad);
  if (bad == 0) return;
  asm volatile("" : "+s"(heads));
  const int lane = ar_lane();
  for (int i = 0; i < 32 && first + i < rows; ++i)
    if (bad >> i & 1) f(first + i, lane, (int)(blockIdx.x % heads), (int)(blockIdx.x / heads));
}
// The sum of ar_probe over a lane's accumulators.
template <int D>
__device__ __forceinline__ float at_probe(const floatx16 (&acc)[AttnCfg<D>::DB], float t) {
#pragma unroll
  for (int db = 0; db < AttnCfg<D>::DB; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) t = ar_probe(t, acc[db][r]);
  return t;
}

// ---------------------------------------------------------------------------
// forward
// ---------------------------------------------------------------------------
template <int D, bool CAUSAL, bool DROP, bool EDGE>
__global__ __launch_bounds__(256, 2) void attn_fwd_mfma_kernel(const bf16* __restrict__ qkv, bf16* __restrict__ ctx,
                                                            float* __restrict__ lse, int s, int heads,
                                                            float scale_log2e, DropArgs drop, int d) {
  using C = AttnCfg<D>;
  __shared__ __attribute__((aligned(16))) bf16 sk[64 * C::PITCH];
  __shared__ __attribute__((aligned(16))) bf16 sv[64 * C::PITCH];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, hf = lane >> 5;
  // Grid: x = (batch, head), y = query block.  Workgroups are dispatched in x-fastest order,
  // so under the causal mask every head's longest (latest) query blocks start first and only
  // short ones are left at the end of the launch; and because consecutive workgroups go round
  // the 8 XCDs, all query blocks of one head (same x mod 8) share one XCD's L2 for K and V.
  const int qb = gridDim.y - 1 - blockIdx.y;
  const int head = blockIdx.x % heads, bi = blockIdx.x / heads;
  const int cols = EDGE ? d : D, h = heads * cols;
  const int64_t ld = 3 * (int64_t)h;
  const bf16* base = qkv + (int64_t)bi * s * ld + head * cols;
  const int q0 = qb * 128, qw = q0 + wave * 32, qw_s = __builtin_amdgcn_readfirstlane(qw);  // this wave's first query
  const int query = qw + (lane & 31);

  const int qrow = EDGE && query >= s ? s - 1 : query;   // queries past the end repeat the last one and are not stored
  bf16x8 qf[C::KD];
  at_load_row<D, EDGE>(qf, base + (int64_t)qrow * ld, hf, cols);

  floatx16 o[C::DB];
#pragma unroll
  for (int i = 0; i < C::DB; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[i][r] = 0.f;
  float m = -INFINITY, l = 0.f;

  const int nkt = (s + 63) / 64, nkb = CAUSAL && (!EDGE || (q0 + 128) / 64 < nkt) ? (q0 + 128) / 64 : nkt;
  AttnTilePair<D, EDGE, 64> rt;   // waves 0 and 1 move the K tile, 2 and 3 the V tile
  const int second = __builtin_amdgcn_readfirstlane(wave >> 1);
  rt.init(base + h + (second ? h : 0), ld, tid & 127, cols);
  rt.load(0, s, cols);
  for (int kb = 0; kb < nkb; ++kb) {
    if (kb) __syncthreads();
    rt.store(second ? sv : sk);
    __syncthreads();
    if (kb + 1 < nkb) rt.load((kb + 1) * 64, s, cols);
    const int k0 = kb * 64;
    if (CAUSAL && k0 > qw_s + 31) continue;  // whole key block is in this wave's future
    // Fragments are fetched a batch of products ahead (left alone, the compiler pairs every read with its product and waits), the
    // first V^T fragments before the last scores are multiplied; the fences keep it that way.
    floatx16 sc[2];
#pragma unroll
    for (int sb = 0; sb < 2; ++sb)
#pragma unroll
      for (int r = 0; r < 16; ++r) sc[sb][r] = 0.f;
    constexpr int KB = D == 96 ? 3 : (D == 32 ? 2 : 4), NB = 2 * C::KD / KB;
    bf16x8 kfr[2][KB], vtr[2][C::DB];
    auto k_frags = [&](int b) {
#pragma unroll
      for (int t = 0; t < KB; ++t) kfr[b & 1][t] = at_row_frag<D>(sk, (b * KB + t) / C::KD * 32, (b * KB + t) % C::KD, lane);
    };
    auto v_frags = [&](int t) {
#pragma unroll
      for (int db = 0; db < C::DB; ++db) vtr[t & 1][db] = at_tr_frag<D>(sv, 16 * t, db * 32, lane);
    };
    k_frags(0);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      if (b + 1 < NB) k_frags(b + 1);
      else v_frags(0);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int t = 0; t < KB; ++t) {
        const int sb = (b * KB + t) / C::KD;
        sc[sb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kfr[b & 1][t], qf[(b * KB + t) % C::KD], sc[sb], 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    v_frags(1);
    __builtin_amdgcn_sched_barrier(0);
    // Raw scores stay in the accumulators until the exponential: the row maximum is taken on
    // them (the scale is positive), and scale and shift fold into one fused multiply-add.
    // Only key blocks that straddle the diagonal pay for the mask.
    float p[2][16];
    float mx = -INFINITY;
    if ((CAUSAL && k0 + 63 > qw_s) || (EDGE && k0 + 64 > s)) {
#pragma unroll
      for (int sb = 0; sb < 2; ++sb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int key = k0 + sb * 32 + 8 * (r >> 2) + 4 * hf + (r & 3);
          if ((CAUSAL && key > query) || (EDGE && key >= s)) sc[sb][r] = -INFINITY;
        }
    }
#pragma unroll
    for (int sb = 0; sb < 2; ++sb)
#pragma unroll
      for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sc[sb][r]);
    // The running reference m only moves when a row's maximum grows by more than 2^8: until
    // then the exponentials are taken against the old reference (they stay below 256, l and
    // the output carry the same factor and the final division removes it), and the block
    // skips rescaling the output accumulators.  Key 0 is visible to every query, so the
    // first block always sets a finite reference.
    // (Each half wave has seen half of a row's scores: only where one of them grows do they compare.)
    if (__builtin_amdgcn_ballot_w64(fmaxf(m, mx * scale_log2e) > m + 8.0f) != 0) {
      const float m_cand = fmaxf(m, fmaxf(mx, __shfl_xor(mx, 32, 64)) * scale_log2e);
      const bool grow = m_cand > m + 8.0f;
      const float m_new = grow ? m_cand : m;
      const float alpha = __builtin_amdgcn_exp2f(m - m_new);
      m = m_new;
      l *= alpha;
#pragma unroll
      for (int i = 0; i < C::DB; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[i][r] *= alpha;
    }
    float psum = 0.f;
#pragma unroll
    for (int sb = 0; sb < 2; ++sb)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        p[sb][r] = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[sb][r], scale_log2e, -m));
        psum += p[sb][r];
      }
    l += psum;   // the softmax is normalised before the dropout
    if (DROP) {
      // this lane's 16 probabilities of a 32-key block are 4 groups of 4 consecutive keys of
      // ONE mask row (its query): one generator call per block, shared within the lane quad
      const uint32_t drow = (uint32_t)(((int64_t)bi * heads + head) * s + query);
#pragma unroll
      for (int sb = 0; sb < 2; ++sb) {
        uint32_t w[4];
        if (EDGE && (s & 3)) at_drop_row_words_any(drop, drow, (uint32_t)(k0 + sb * 32 + 4 * hf) >> 2, w);
        else at_drop_row_words(drop, drow >> 2, (uint32_t)(k0 + sb * 32 + 4 * hf) >> 2, lane, w);
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (!drop_keep(drop, w[g], e)) p[sb][4 * g + e] = 0.f;
      }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const bf16x8 pf = at_pack8(&p[t >> 1][8 * (t & 1)]);
#pragma unroll
      for (int db = 0; db < C::DB; ++db)
        o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vtr[t & 1][db], pf, o[db], 0, 0, 0);
      if constexpr (EDGE) {
        const bf16x8 pl = at_pack8_rest(&p[t >> 1][8 * (t & 1)], pf);
#pragma unroll
        for (int db = 0; db < C::DB; ++db)
          o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vtr[t & 1][db], pl, o[db], 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
      if (t < 2) v_frags(t + 2);   // into the registers just multiplied
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  l += __shfl_xor(l, 32, 64);
  const float inv = (DROP ? drop.scale : 1.0f) / l;
  const uint32_t bad = EDGE ? ar_bad_rows(at_probe<D>(o, ar_probe(0.f, l))) : 0;   // rows that are not finite: below
  if (!EDGE || (query < s && !(bad >> (ar_lane() & 31) & 1))) {
    if (lse && hf == 0) {
      float& out = lse[((int64_t)bi * heads + head) * s + query];
      if constexpr (EDGE) out = (float)(((double)m + (double)log2f(l)) * 0.69314718055994531);   // one rounding, as the natural logarithm of a row kernel
      else out = (m + log2f(l)) * 0.6931471805599453f;
    }
    bf16* crow = ctx + ((int64_t)bi * s + query) * h + head * cols;
#pragma unroll
    for (int db = 0; db < C::DB; ++db)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        if (EDGE && db * 32 + 8 * g >= cols) continue;
        bf16x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = (bf16)(o[db][4 * g + e] * inv);
        *reinterpret_cast<bf16x4*>(crow + db * 32 + 8 * g + 4 * hf) = v;
      }
  }
  if constexpr (EDGE) at_bad_rows(bad, qw_s, s, heads, [&](int i, int ln, int hd, int b) {
    const int64_t at = (int64_t)b * s * heads * d + hd * d;
    ar_fwd<bf16>(qkv + 3 * at - 2 * hd * d, ctx + at, lse, i, s, heads * d, d, CAUSAL, 1.0f / sqrtf((float)d), ((int64_t)b * heads + hd) * s, drop, ln);
  });
}

// ---------------------------------------------------------------------------
// backward, query side: dQ and delta
// ---------------------------------------------------------------------------
template <int D, bool CAUSAL, bool DROP, bool EDGE>
__global__ __launch_bounds__(256, 2) void attn_bwd_dq_mfma_kernel(const bf16* __restrict__ qkv, const bf16* __restrict__ ctx,
                                                               const float* __restrict__ lse,
                                                               const bf16* __restrict__ dctx, bf16* __restrict__ dqkv,
                                                               float* __restrict__ delta, int s, int heads,
                                                               float scale, float scale_log2e, DropArgs drop, int d) {
  using C = AttnCfg<D>;
  __shared__ __attribute__((aligned(16))) bf16 sk[64 * C::PITCH];
  __shared__ __attribute__((aligned(16))) bf16 sv[64 * C::PITCH];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, hf = lane >> 5;
  const int qb = gridDim.y - 1 - blockIdx.y;   // grid as in the forward kernel: long query blocks of every head first
  const int head = blockIdx.x % heads, bi = blockIdx.x / heads;
  const int cols = EDGE ? d : D, h = heads * cols;
  const int64_t ld = 3 * (int64_t)h;
  const bf16* base = qkv + (int64_t)bi * s * ld + head * cols;
  const int q0 = qb * 128, qw = q0 + wave * 32, qw_s = __builtin_amdgcn_readfirstlane(qw);
  const int query = qw + (lane & 31);
  const int qrow = EDGE && query >= s ? s - 1 : query;   // queries past the end repeat the last one and store nothing
  const int64_t orow = ((int64_t)bi * s + qrow) * h + head * cols;
  const int64_t sidx = ((int64_t)bi * heads + head) * s + qrow;

  bf16x8 qf[C::KD], gf[C::KD];
  float dl = 0.f;
  {
    bf16x8 of[C::KD];
    at_load_row<D, EDGE>(qf, base + (int64_t)qrow * ld, hf, cols);
    at_load_row<D, EDGE>(gf, dctx + orow, hf, cols);
    at_load_row<D, EDGE>(of, ctx + orow, hf, cols);
#pragma unroll
    for (int t = 0; t < C::KD; ++t)
#pragma unroll
      for (int e = 0; e < 8; ++e) dl += (float)gf[t][e] * (float)of[t][e];
  }
  dl += __shfl_xor(dl, 32, 64);
  if (hf == 0 && (!EDGE || query < s)) delta[sidx] = dl;
  const float l2 = lse[sidx] * 1.4426950408889634f;  // log-sum-exp in base 2

  floatx16 dq[C::DB];
#pragma unroll
  for (int i = 0; i < C::DB; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) dq[i][r] = 0.f;

  const int nkt = (s + 63) / 64, nkb = CAUSAL && (!EDGE || (q0 + 128) / 64 < nkt) ? (q0 + 128) / 64 : nkt;
  AttnTilePair<D, EDGE, 64> rt;   // waves 0 and 1 move the K tile, 2 and 3 the V tile
  const int second = __builtin_amdgcn_readfirstlane(wave >> 1);
  rt.init(base + h + (second ? h : 0), ld, tid & 127, cols);
  rt.load(0, s, cols);
  for (int kb = 0; kb < nkb; ++kb) {
    if (kb) __syncthreads();
    rt.store(second ? sv : sk);
    __syncthreads();
    if (kb + 1 < nkb) rt.load((kb + 1) * 64, s, cols);
    const int k0 = kb * 64;
    // (no per-wave skip of key blocks in this wave's future: the mask zeroes them, and a
    // branch around the products costs registers)
    const bool need_mask = (CAUSAL && k0 + 63 > qw_s) || (EDGE && k0 + 64 > s);
    // Fragments are fetched a batch ahead of their products, across the two halves of the tile (see the forward kernel).
    constexpr int KB = D == 96 ? 3 : (D == 128 && DROP && !EDGE ? 1 : 2), NB = C::KD / KB;
    bf16x8 kfr[2][KB], vfr[2][KB], ktr[2][C::DB];
    auto rows = [&](int sb, int b) {
#pragma unroll
      for (int t = 0; t < KB; ++t) {
        kfr[b & 1][t] = at_row_frag<D>(sk, sb * 32, b * KB + t, lane);
        vfr[b & 1][t] = at_row_frag<D>(sv, sb * 32, b * KB + t, lane);
      }
    };
    auto k_cols = [&](int sb, int t) {
#pragma unroll
      for (int db = 0; db < C::DB; ++db) ktr[t][db] = at_tr_frag<D>(sk, sb * 32 + 16 * t, db * 32, lane);
    };
    if (D < 128) rows(0, 0);
#pragma unroll
    for (int sb = 0; sb < 2; ++sb) {
      floatx16 sc, dp;
#pragma unroll
      for (int r = 0; r < 16; ++r) { sc[r] = 0.f; dp[r] = 0.f; }
      if (D == 128) rows(sb, 0);
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        if (b + 1 < NB) rows(sb, b + 1);
        else k_cols(sb, 0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < KB; ++t) {
          sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kfr[b & 1][t], qf[b * KB + t], sc, 0, 0, 0);
          dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vfr[b & 1][t], gf[b * KB + t], dp, 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if (DROP) {  // dP = dropout'(dO V^T): same mask words as the forward kernel
        uint32_t w[4];
        // (a query past the end must not take its quad to another row of patches: it stores nothing, so any word serves)
        const uint32_t drow = (uint32_t)(((int64_t)bi * heads + head) * s + query);
        if (EDGE && (s & 3)) at_drop_row_words_any(drop, drow, (uint32_t)(k0 + sb * 32 + 4 * hf) >> 2, w);
        else at_drop_row_words(drop, drow >> 2, (uint32_t)(k0 + sb * 32 + 4 * hf) >> 2, lane, w);
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
          for (int e = 0; e < 4; ++e) dp[4 * g + e] = drop_keep(drop, w[g], e) ? dp[4 * g + e] * drop.scale : 0.f;
      }
      if (need_mask) {   // blocks that straddle or follow the diagonal, or the end of the sequence
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int key = k0 + sb * 32 + 8 * (r >> 2) + 4 * hf + (r & 3);
          if ((CAUSAL && key > query) || (EDGE && key >= s)) sc[r] = -INFINITY;
        }
      }
      float ds[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float pr = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[r], scale_log2e, -l2));
        ds[r] = pr * (dp[r] - dl);
      }
      __builtin_amdgcn_sched_barrier(0);
      k_cols(sb, 1);
      if (D < 128 && sb == 0) rows(1, 0);   // (at d = 128 there is no register left for it)
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const bf16x8 df = at_pack8(&ds[8 * t]);
#pragma unroll
        for (int db = 0; db < C::DB; ++db)
          dq[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ktr[t][db], df, dq[db], 0, 0, 0);
        if constexpr (EDGE) {
          const bf16x8 dl8 = at_pack8_rest(&ds[8 * t], df);
#pragma unroll
          for (int db = 0; db < C::DB; ++db)
            dq[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ktr[t][db], dl8, dq[db], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  const uint32_t bad = EDGE ? ar_bad_rows(at_probe<D>(dq, 0.f)) : 0;
  if (!EDGE || (query < s && !(bad >> (ar_lane() & 31) & 1))) {
    bf16* drow = dqkv + ((int64_t)bi * s + query) * ld + head * cols;
#pragma unroll
    for (int db = 0; db < C::DB; ++db)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        if (EDGE && db * 32 + 8 * g >= cols) continue;
        bf16x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = (bf16)(dq[db][4 * g + e] * scale);
        *reinterpret_cast<bf16x4*>(drow + db * 32 + 8 * g + 4 * hf) = v;
      }
  }
  if constexpr (EDGE) at_bad_rows(bad, qw_s, s, heads, [&](int i, int ln, int hd, int b) {
    const int64_t at = (int64_t)b * s * heads * d + hd * d, at3 = 3 * at - 2 * hd * d;
    ar_dq<bf16>(qkv + at3, ctx + at, dctx + at, lse, dqkv + at3, i, s, heads * d, d, CAUSAL, scale, ((int64_t)b * heads + hd) * s, drop, ln);
  });
}

// ---------------------------------------------------------------------------
// backward, key side: dK and dV
// ---------------------------------------------------------------------------
// Waves per SIMD.  Two waves have 256 registers each: dK, dV, K and V of 32 keys are 96 (d = 64) to 192 (d = 128) of them.  The
// forms whose masks or second parts of P and dS do not fit run on one wave with twice the registers; a spill is worse (its reload waits
// for the next tile's loads: 64 heads of 128 over 2048 tokens, causal, 8 registers spilled 180 us, none 130).
constexpr int attn_dkv_waves(int d, bool drop, bool edge) { return (edge && d == 128) || (drop && (d == 128 || (edge && d == 96))) ? 1 : 2; }
// 32 queries per step, two stages, one barrier per step.  From the last queries to the first: under the causal mask the key blocks
// of a head, which start together, then read the same tiles at the same time.
//
// us for dQ, dK and dV against the form on one wave per SIMD that fetched 64-query tiles through 64-bit addresses: 64 heads of 128
// over 2048 tokens 350 / 254, 80 of 96 over 1024 123 / 90 (all causal), 128 of 64 over 512 47 / 45, 50 of 64 over 1000 (EDGE) 87 / 65.
template <int D, bool CAUSAL, bool DROP, bool EDGE>
__global__ __launch_bounds__(256, attn_dkv_waves(D, DROP, EDGE)) void attn_bwd_dkv_mfma_kernel(const bf16* __restrict__ qkv, const float* __restrict__ lse,
                                                                const bf16* __restrict__ dctx,
                                                                const float* __restrict__ delta, bf16* __restrict__ dqkv,
                                                                int s, int heads, float scale, float scale_log2e,
                                                                DropArgs drop, int d) {
  using C = AttnCfg<D>;
  constexpr int TILE = 32 * C::PITCH;
  // At d = 128 two waves have no registers for V: its fragments, and the first of K, are kept in LDS (each wave's own).
  constexpr bool VLDS = D == 128 && attn_dkv_waves(D, DROP, EDGE) == 2;
  __shared__ __attribute__((aligned(16))) bf16 sqg[2][2][TILE];   // [stage][Q, dO]
  __shared__ __attribute__((aligned(16))) bf16x8 svf[VLDS ? 4 * (C::KD + 1) * 64 : 1];
  __shared__ __attribute__((aligned(16))) float sstat[2][2][32];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), hf = lane >> 5;
  // grid: x = (batch, head), y = key block; early key blocks (most queries under the causal
  // mask) of every head are dispatched first
  const int kblk = blockIdx.y;
  const int head = blockIdx.x % heads, bi = blockIdx.x / heads;
  const int cols = EDGE ? d : D, h = heads * cols;
  const int64_t ld = 3 * (int64_t)h;
  const bf16* base = qkv + (int64_t)bi * s * ld + head * cols;
  const bf16* gbase = dctx + (int64_t)bi * s * h + head * cols;
  const int kb0 = kblk * 128, kw = kb0 + wave * 32;  // this wave's first key
  const int key = kw + (lane & 31);
  const int64_t sbase = ((int64_t)bi * heads + head) * s;

  const int key_row = EDGE && key >= s ? s - 1 : key;   // keys past the end repeat the last one and are not stored
  bf16x8 kf[C::KD], vf[C::KD];
  at_load_row<D, EDGE>(kf, base + (int64_t)key_row * ld + h, hf, cols);
  at_load_row<D, EDGE>(vf, base + (int64_t)key_row * ld + 2 * h, hf, cols);
  bf16x8* svw = svf + (VLDS ? wave * (C::KD + 1) * 64 + lane : 0);
  if constexpr (VLDS) {
#pragma unroll
    for (int t = 0; t < C::KD; ++t) svw[t * 64] = vf[t];
    svw[C::KD * 64] = kf[0];
  }
  floatx16 dk[C::DB], dv[C::DB];
#pragma unroll
  for (int i = 0; i < C::DB; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) { dk[i][r] = 0.f; dv[i][r] = 0.f; }

  const int qs = CAUSAL ? kb0 / 32 : 0, nqb = (s + 31) / 32;
  AttnTilePair<D, EDGE, 32> rt;   // waves 0 and 1 move the Q tile, 2 and 3 the dO tile
  const int second = wave >> 1;
  rt.init(second ? gbase : base, second ? (int64_t)h : ld, tid & 127, cols);
  // Waves 0 and 1 also carry the tile's lse and delta (zero for queries past the end, whose rows of Q and dO are zero: EDGE, where the whole
  // offset is the part that the range check sees, as in AttnTilePair).
  float rstat = 0.f;
  [[maybe_unused]] const float* stats = (wave == 0 ? lse : delta) + sbase;
  auto load = [&](int qb) {
    rt.load(qb * 32, s, cols);
#if defined(__HIP_DEVICE_COMPILE__)
    if (wave < 2) rstat = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(__builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(stats), 0, s * 4, 0x00020000), (lane & 31) * 4 + (EDGE ? qb * 128 : 0), EDGE ? 0 : qb * 128, 0));
#endif
  };
  auto store = [&](int st) {
    rt.store(sqg[st][second]);
    if (wave < 2 && lane < 32) sstat[st][wave][lane] = wave == 0 ? rstat * 1.4426950408889634f : -rstat;
  };
  load(nqb - 1);
  store((nqb - 1) & 1);
  __syncthreads();
  for (int qb = nqb - 1; qb >= qs; --qb) {
    const int st = qb & 1;
    if (qb > qs) load(qb - 1);
    const int q0 = qb * 32;
    if (!CAUSAL || q0 + 31 >= kw) {   // else every key of this wave follows the tile's queries
      const bool need_mask = CAUSAL && (q0 < kw + 31);
      const bf16* tq = sqg[st][0];
      const bf16* tg = sqg[st][1];
      // Fragments are fetched a batch of products ahead; the fences keep the order (see the forward kernel).
      constexpr int KB = D == 128 || (EDGE && D == 96) ? 1 : 2;
      bf16x8 qfr[2][KB], gfr[2][KB], vfr[2][KB];
      auto fetch = [&](int b) {
#pragma unroll
        for (int t = 0; t < KB; ++t) {
          qfr[b & 1][t] = at_row_frag<D>(tq, 0, b * KB + t, lane);
          gfr[b & 1][t] = at_row_frag<D>(tg, 0, b * KB + t, lane);
          if constexpr (VLDS) vfr[b & 1][t] = svw[(b * KB + t) * 64];
        }
      };
      floatx16 sc, dp;
#pragma unroll
      for (int r = 0; r < 16; ++r) { sc[r] = 0.f; dp[r] = DROP ? 0.f : sstat[st][1][8 * (r >> 2) + 4 * hf + (r & 3)]; }   // dP - delta in one sum
      constexpr int NB = C::KD / KB;
      fetch(0);
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        if (b + 1 < NB) fetch(b + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < KB; ++t) {
          sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qfr[b & 1][t], VLDS && b * KB + t == 0 ? svw[C::KD * 64] : kf[b * KB + t], sc, 0, 0, 0);
          dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(gfr[b & 1][t], VLDS ? vfr[b & 1][t] : vf[b * KB + t], dp, 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      // The last products' column operands, pair number k = (16 queries t, block db): PF pairs in flight.
      constexpr int NP = 2 * C::DB, PF = EDGE ? (D == 96 ? 1 : 2) : (D == 96 && !DROP ? 3 : (D >= 96 ? 2 : NP));
      bf16x8 gtr[PF], qtr[PF];
      auto cols_of = [&](int k) {
        gtr[k % PF] = at_tr_frag<D>(tg, 16 * (k / C::DB), k % C::DB * 32, lane);
        qtr[k % PF] = at_tr_frag<D>(tq, 16 * (k / C::DB), k % C::DB * 32, lane);
      };
#pragma unroll
      for (int k = 0; k < PF; ++k) cols_of(k);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const floatx4 l4 = *reinterpret_cast<const floatx4*>(&sstat[st][0][8 * g + 4 * hf]);
#pragma unroll
        for (int e = 0; e < 4; ++e) sc[4 * g + e] = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[4 * g + e], scale_log2e, -l4[e]));
      }
      if (need_mask) {   // tiles that straddle the diagonal; after the exponential: a masked query's log-sum-exp may be a NaN
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (q0 + 8 * (r >> 2) + 4 * hf + (r & 3) < key) sc[r] = 0.f;
      }
      float pr[16], ds[16];
      uint32_t own[4];
      const bool patches = DROP && !(EDGE && (s & 3));   // groups of 4 queries are rows of patches
      if (patches) drop_patch(drop, ((uint32_t)(sbase + q0 + 4 * hf) >> 2) + 2u * (uint32_t)(lane & 3), (uint32_t)key >> 2, own);
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int ql = 8 * g + 4 * hf;  // 4 consecutive queries of the tile
        floatx4 d4 = {0.f, 0.f, 0.f, 0.f};
        if (DROP) d4 = *reinterpret_cast<const floatx4*>(&sstat[st][1][ql]);
        uint32_t mw[4];
        if (patches) {
#pragma unroll
          for (int e = 0; e < 4; ++e) mw[e] = at_quad_bcast(own[e], g);
        } else if (DROP) {
#pragma unroll
          for (int e = 0; e < 4; ++e) mw[e] = drop_row_word(drop, (uint32_t)(sbase + q0 + ql + e), (uint32_t)key >> 2);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int r = 4 * g + e;
          float f = 1.0f;
          if (DROP) f = drop_keep(drop, mw[e], key & 3) ? drop.scale : 0.f;
          pr[r] = sc[r] * f;
          ds[r] = DROP ? sc[r] * (dp[r] * f + d4[e]) : sc[r] * dp[r];
        }
      }
      bf16x8 pf, df, pl, dl;
#pragma unroll
      for (int k = 0; k < NP; ++k) {
        const int t = k / C::DB, db = k % C::DB;
        if (db == 0) {
          pf = at_pack8(&pr[8 * t]);
          df = at_pack8(&ds[8 * t]);
          if constexpr (EDGE) { pl = at_pack8_rest(&pr[8 * t], pf); dl = at_pack8_rest(&ds[8 * t], df); }
        }
        dv[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(gtr[k % PF], pf, dv[db], 0, 0, 0);
        dk[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qtr[k % PF], df, dk[db], 0, 0, 0);
        if constexpr (EDGE) {
          dv[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(gtr[k % PF], pl, dv[db], 0, 0, 0);
          dk[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qtr[k % PF], dl, dk[db], 0, 0, 0);
        }
        if (k + PF < NP) cols_of(k + PF);   // into the registers just multiplied
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (qb > qs) store(st ^ 1);
    __syncthreads();
  }
  const uint32_t bad = EDGE ? ar_bad_rows(at_probe<D>(dk, at_probe<D>(dv, 0.f))) : 0;
  if (!EDGE || (key < s && !(bad >> (ar_lane() & 31) & 1))) {
    bf16* krow = dqkv + ((int64_t)bi * s + key) * ld + h + head * cols;
    bf16* vrow = krow + h;
#pragma unroll
    for (int db = 0; db < C::DB; ++db)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        if (EDGE && db * 32 + 8 * g >= cols) continue;
        bf16x4 a, c;
#pragma unroll
        for (int e = 0; e < 4; ++e) { a[e] = (bf16)(dk[db][4 * g + e] * scale); c[e] = (bf16)dv[db][4 * g + e]; }
        *reinterpret_cast<bf16x4*>(krow + db * 32 + 8 * g + 4 * hf) = a;
        *reinterpret_cast<bf16x4*>(vrow + db * 32 + 8 * g + 4 * hf) = c;
      }
  }
  if constexpr (EDGE) at_bad_rows(bad, kw, s, heads, [&](int i, int ln, int hd, int b) {
    const int64_t at = (int64_t)b * s * heads * d + hd * d, at3 = 3 * at - 2 * hd * d;
    ar_dkv<bf16>(qkv + at3, dctx + at, lse, delta, dqkv + at3, i, s, heads * d, d, CAUSAL, scale, ((int64_t)b * heads + hd) * s, drop, ln);
  });
}

}  // namespace varuna
