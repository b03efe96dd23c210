// GEMM of fp32 accuracy on the bf16 matrix cores: acc[m,n] = sum_k A(m,k) * B(n,k), any M, N, K.
//   AK: A(m,k) = a[m*lda + k]   else A(m,k) = a[k*lda + m];   BK likewise for B(n,k) = b[n*ldb + k] / b[k*ldb + n]
// It takes the bf16 operands whose rows are not whole 16-byte pieces (the direct-to-LDS kernels cannot address them), bf16 products of few
// tiles (dg_cut_sooner), and those fp32 products where it is faster than the fp32 matrix instructions of gemm_f32.h (gc_kind).
//
// An fp32 operand is cut into three bf16 pieces, x = x1 + x2 + x3 with x1 = bf16(x), x2 = bf16(x - x1), x3 = the rest: 24 bits of
// mantissa in pieces of 8, nothing is left over.  Of the nine piece products six are summed in fp32 (x1y1, x1y2, x2y1, x2y2, x1y3, x3y1),
// x1y1 in a sum of its own: a sum rounds relative to its size.  Left out are x2y3 + x3y2, at worst 2^-24 of a product, half a unit of an fp32
// result (near 1.004 times 1.004; a tenth of that on average, of either sign), and x3y3, 2^-34.  A single product shows that (8.8e-8 off
// where an fp32 product is 6.0e-8), a sum of 128 and more, the shortest that comes here, does not: operands within 1e-5 of that worst
// place over K = 200 / 300 / 1024 / 3072 are 3.7e-8 / 2.9e-8 / 5.0e-8 / 3.9e-8 from 64 bits with these six as with eight of the products, in
// fp32 products 2.1e-7 / 2.5e-7 / 2.8e-7 / 1.1e-7; eight take 8 to 13 % longer ([1000,768] over 3072 43 -> 48 us, 2048^3 123 -> 140).
// N(0,1) operands, fp32 products / this (K = 301, 1024, 3072, 2048 on one wave): 1.3e-7 / 7.1e-8, 5.7e-7 / 9.8e-8, 3.6e-7 / 1.6e-7,
// 8.1e-7 / 2.7e-7.  A bf16 operand is its own only piece.
//
// What bounds it: fp32, the vector instructions that cut (seven and a half per element and wave) beside products at the rate real data
// sustains; bf16, the path from L2 (16 KB per 64x64x64 block).  Every wave works alone, on its own steps of the reduction: no
// barrier until the sums meet, and the cutting of one step issues between the products of the step before.  Reading the
// operands straight into registers instead (32 rows of 32 bytes per instruction) took 1.2 to 3 times as long: one cache line per
// clock; sharing cut tiles through LDS between waves was equal at 2048^3 and slower below.  Measured (us, fp32 products / this):
// bf16 [4001,3001] over 3001 1515 / 246, 1001^3 65 / 12, 301^3 8.9 / 4.3; fp32 [1000,768] over 3072 57 / 44, 2048^3 154 / 120,
// 1024^3 27 / 21, [512,512] over 2048 17.3 / 14.2.
#pragma once
#include <type_traits>

#include "common.h"
#include "gemm_epilogue.h"
#include "gemm_f32.h"

namespace varuna {

template <typename T> struct GcPieces { static constexpr int N = 1; };
template <> struct GcPieces<float> { static constexpr int N = 3; };

typedef uint32_t gc_words __attribute__((ext_vector_type(4)));

// Eight consecutive k of one row as the operand of a 32x32x16 product, in NP pieces.
template <typename T> struct GcFrag { bf16x8 p[GcPieces<T>::N]; };

__device__ __forceinline__ GcFrag<bf16> gc_cut(const gc_words& x, uint32_t&) { return {{__builtin_bit_cast(bf16x8, x)}}; }
// lost: every bit of the rests is or-ed into it; the lower 16 are what the third pieces leave out (gc_exact_block).
__device__ __forceinline__ GcFrag<float> gc_cut(const float (&x)[8], uint32_t& lost) {
  gc_words h, m, l;   // two pieces per word
#pragma unroll
  for (int e = 0; e < 8; e += 2) {
    const bf16x2 hp = {(bf16)x[e], (bf16)x[e + 1]};
    uint32_t hw = __builtin_bit_cast(uint32_t, hp);
    asm("" : "+v"(hw));   // (seen through, the first half is converted a second time)
    const float y0 = x[e] - __builtin_bit_cast(float, hw << 16), y1 = x[e + 1] - __builtin_bit_cast(float, hw & 0xffff0000u);
    const bf16x2 mp = {(bf16)y0, (bf16)y1};
    uint32_t mw = __builtin_bit_cast(uint32_t, mp);
    asm("" : "+v"(mw));
    const float z0 = y0 - __builtin_bit_cast(float, mw << 16), z1 = y1 - __builtin_bit_cast(float, mw & 0xffff0000u);
    h[e / 2] = hw;
    m[e / 2] = mw;
    const uint32_t zw0 = __builtin_bit_cast(uint32_t, z0), zw1 = __builtin_bit_cast(uint32_t, z1);
    l[e / 2] = __builtin_amdgcn_perm(zw1, zw0, 0x07060302u);   // upper halves: all there is from 2^-109 on
    lost |= zw0 | zw1;
  }
  GcFrag<float> f;
  f.p[0] = __builtin_bit_cast(bf16x8, h); f.p[1] = __builtin_bit_cast(bf16x8, m); f.p[2] = __builtin_bit_cast(bf16x8, l);
  return f;
}

// One operand of a wave: NB blocks of 32 rows, steps of 64 bytes of k (fp32: 16 k, bf16: 32).  A step goes from memory into registers in
// whole 16-byte pieces (rows of 64 bytes, or k-rows of all the rows), through the wave's own part of LDS and back in the layout
// of a product's operand: lane l holds row l % 32 of every block and k 8 * (l / 32) .. +7 of a 16-k group.  KMAJOR: block i, row r is
// row 32 i + r of the tile, 16-byte pieces XOR-permuted by row / 4 so that a read's 16 rows fall into different banks; else row
// NB r + i, so that a lane's rows are neighbours.
template <typename T, int NB, bool KMAJOR>
struct GcOperand {
  static constexpr int EPP = 16 / sizeof(T), KST = 4 * EPP, ROWS = 32 * NB, PIECES = ROWS * 4 / kWave;   // pieces of a lane per step
  static constexpr int BYTES = ROWS * 64, PPK = ROWS / EPP;   // n-major: pieces of a k-row
  // bf16 elements are held two per word throughout: as elements the compiler gives each a register of its own.
  typedef std::conditional_t<sizeof(T) == 4, float, uint32_t> Word;
  typedef Word Piece __attribute__((ext_vector_type(4), aligned(sizeof(T))));   // (element-aligned is enough)
  typedef Word PieceA __attribute__((ext_vector_type(4)));
  struct Raw { PieceA v[PIECES]; };
  struct Group { std::conditional_t<sizeof(T) == 4, float[8], gc_words> v[NB]; };   // a 16-k group of every block
  const T* p[PIECES];      // this lane's pieces of step 0
  int64_t kpitch;          // elements from one k to the next

  static __device__ __forceinline__ int row(int i, int r) { return KMAJOR ? 32 * i + r : NB * r + i; }
  static __device__ __forceinline__ int piece_line(int q, int lane) { return KMAJOR ? q * 16 + lane / 4 : q * (kWave / PPK) + lane / PPK; }   // row, or k
  static __device__ __forceinline__ int piece_elem(int q, int lane) {   // first k of the piece, or first row
    if constexpr (KMAJOR) return ((lane & 3) ^ (piece_line(q, lane) >> 2 & 3)) * EPP;
    else return lane % PPK * EPP;
  }
  __device__ __forceinline__ void init(const T* __restrict__ g, int64_t ld, int64_t row0, int64_t rows, int lane) {
    kpitch = KMAJOR ? 1 : ld;
    // Rows past the end (nothing of them is stored) repeat the last one, or the last whole piece of a k-row; of a k-row that does not end
    // with a whole piece they are the last row and what follows it in memory, which `over` in GcTile keeps inside the operand.
    const int64_t end = KMAJOR || rows % EPP != 0 ? rows - 1 : rows - EPP;
#pragma unroll
    for (int q = 0; q < PIECES; ++q) {
      int64_t r = row0 + (KMAJOR ? piece_line(q, lane) : piece_elem(q, lane));
      r = r < rows ? r : end;
      p[q] = KMAJOR ? g + r * ld + piece_elem(q, lane) : g + piece_line(q, lane) * ld + r;
    }
  }
  __device__ __forceinline__ void load(Raw& x, int64_t k) const {
#pragma unroll
    for (int q = 0; q < PIECES; ++q) x.v[q] = *reinterpret_cast<const Piece*>(p[q] + k * kpitch);
  }
  // The last steps: k past the end reads as zero, and no piece runs over its k-row.
  // WHOLE: with a way of its own for rows that are whole pieces (one wave for a 64x64 tile has no registers for it).
  template <bool WHOLE>
  __device__ __forceinline__ void load_last(Raw& x, int64_t k, int64_t K, int64_t row0, int64_t rows, int lane) const {
    if constexpr (!KMAJOR && WHOLE) {
      if (rows % EPP == 0) {   // only k may be past the end, and reads the last k-row in its place
#pragma unroll
        for (int q = 0; q < PIECES; ++q) {
          const int64_t left = K - k - piece_line(q, lane);
          const PieceA t = *reinterpret_cast<const Piece*>(p[q] + (left > 0 ? k : k + left - 1) * kpitch);
          x.v[q] = left > 0 ? t : PieceA{};
        }
        return;
      }
    }
#pragma unroll
    for (int q = 0; q < PIECES; ++q) {
      const int64_t left = K - k - (KMAJOR ? piece_elem(q, lane) : piece_line(q, lane));   // k from the piece's first on
      const int64_t r = row0 + piece_elem(q, lane), last = r < rows ? rows - 1 - r : 0;
      const T* base = p[q] + (KMAJOR || left > 0 ? k : k + left - 1) * kpitch;             // n-major: past the end the last k-row
      auto element = [&](int e) -> T {
        if constexpr (KMAJOR) return e < left ? base[e] : (T)0.f;
        const T v = base[e < last ? e : last];   // (no branch, and a piece at a time: all at once took the registers of a second wave)
        return left > 0 ? v : (T)0.f;
      };
      T t __attribute__((ext_vector_type(EPP)));
#pragma unroll
      for (int e = 0; e < EPP; ++e) t[e] = element(e);
      x.v[q] = __builtin_bit_cast(PieceA, t);
      if constexpr (!KMAJOR) __builtin_amdgcn_sched_barrier(0);
    }
  }
  __device__ __forceinline__ void put(const Raw& x, char* lds, int lane) const {
#pragma unroll
    for (int q = 0; q < PIECES; ++q) *reinterpret_cast<PieceA*>(lds + (q * kWave + lane) * 16) = x.v[q];
  }
  // Group c of the step.
  __device__ __forceinline__ void get(Group& g, const char* lds, int c, int lane) const {
    const int half = lane >> 5, r = lane & 31;
    if constexpr (KMAJOR) {
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int q = 0; q < 8 / EPP; ++q) {
          const int piece = (c * 16 + 8 * half) / EPP + q;
          reinterpret_cast<PieceA*>(&g.v[i])[q] = *reinterpret_cast<const PieceA*>(lds + (i * 32 + r) * 64 + ((piece ^ (r >> 2 & 3)) * 16));
        }
    } else {
      const T* s = reinterpret_cast<const T*>(lds) + (c * 16 + 8 * half) * ROWS + NB * r;
      if constexpr (sizeof(T) == 4) {
        typedef float Rows __attribute__((ext_vector_type(NB)));
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          if constexpr (NB == 1) g.v[0][e] = s[e * ROWS];
          else {
            const Rows t = *reinterpret_cast<const Rows*>(s + e * ROWS);
#pragma unroll
            for (int i = 0; i < NB; ++i) g.v[i][e] = t[i];
          }
        }
      } else {
        static_assert(NB <= 2, "a word holds the rows of a lane");
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const T* s0 = s + 2 * w * ROWS;
          const T* s1 = s0 + ROWS;
          if constexpr (NB == 1) {
            g.v[0][w] = *reinterpret_cast<const uint16_t*>(s0) | (uint32_t)*reinterpret_cast<const uint16_t*>(s1) << 16;
          } else {
            const uint32_t t0 = *reinterpret_cast<const uint32_t*>(s0), t1 = *reinterpret_cast<const uint32_t*>(s1);
            g.v[0][w] = __builtin_amdgcn_perm(t1, t0, 0x05040100u);
            g.v[1][w] = __builtin_amdgcn_perm(t1, t0, 0x07060302u);
          }
        }
      }
    }
  }
};

// One 32x32 block over the steps of wave `ks`, with fp32 products from memory: for sums whose pieces are no good.  An infinity, or a value
// that rounds to one, has NaN as its rest.  Below 2^-109 a value's last bits lie below the smallest bf16, 2^-133 (the matrix cores keep
// bf16 and fp32 denormals): one such operand is enough, as its sums may be as large as any.  And sums of products below 2^-100 reach
// into the denormals with their small terms.  Measured: 2048^3 125 us, with one such row in A 400 (as long as with every row
// such, since all of a round wait for its tiles), 1024^3 23 and 53; the notice taken of it costs 1 to 4 % of a product.
template <bool KMAJOR>
__device__ __forceinline__ void gc_exact_load(float (&x)[8], const float* p, int64_t ld, int64_t k, int64_t K) {   // p: this lane's row
  typedef float Four __attribute__((ext_vector_type(4), aligned(4)));
  if (KMAJOR && k + 8 <= K) {
    const Four lo = *reinterpret_cast<const Four*>(p + k), hi = *reinterpret_cast<const Four*>(p + k + 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) { x[e] = lo[e]; x[4 + e] = hi[e]; }
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int64_t kr = k + e < K ? k + e : K - 1;   // (no branch: the loads are in flight together)
      const float v = KMAJOR ? p[kr] : p[kr * ld];
      x[e] = k + e < K ? v : 0.f;
    }
  }
}
template <bool AK, bool BK>
__device__ __attribute__((noinline)) floatx16 gc_exact_block(const float* a, const float* b, int64_t lda, int64_t ldb, int64_t K, int ks, int nks) {
  constexpr int step = 16;
  const int half = (threadIdx.x % kWave) >> 5;
  floatx16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  for (int64_t s = (int64_t)ks * step; s < K; s += step * nks) {
    float x[8], y[8];   // half 0 has the first eight k of a step, half 1 the others
    gc_exact_load<AK>(x, a, lda, s + 8 * half, K);
    gc_exact_load<BK>(y, b, ldb, s + 8 * half, K);
#pragma unroll
    for (int e = 0; e < 8; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x[e], y[e], acc, 0, 0, 0);
  }
  return acc;
}

// LDS accesses of one wave are served in order; this keeps the compiler from exchanging one lane's write with another's read.
__device__ __forceinline__ void gc_wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_sched_barrier(0);
}

template <int V> struct GcInt { static constexpr int v = V; };

// One workgroup: a 32 TM x 32 TN tile; its KS waves take every KS-th step of k of the whole tile.
template <typename T, int MODE, bool AK, bool BK, int TM, int TN, int KS>
struct GcTile {
  static constexpr int BM = 32 * TM, BN = 32 * TN, NT = KS * kWave, NP = GcPieces<T>::N;
  static constexpr bool PARTS = NP == 1 && (MODE == EPI_ACCUM_F32 || MODE == EPI_STORE_F32);
  using OA = GcOperand<T, TM, AK>;
  using OB = GcOperand<T, TN, BK>;
  static constexpr int KST = OA::KST, GROUPS = KST / 16, STAGE = OA::BYTES + OB::BYTES;
  static constexpr size_t RED = KS > 1 ? sizeof(float) * KS * TM * TN * 1024 : 0, RING = (size_t)KS * 2 * STAGE, SMEM = RED > RING ? RED : RING;

  static __device__ __forceinline__ void run(const T* __restrict__ a, int64_t lda, const T* __restrict__ b, int64_t ldb, int64_t M,
                                             int64_t N, int64_t K, int tiles_m, int tiles_n, const EpiArgs<T>& epi, int logical, float* red) {
    const int tid = threadIdx.x, lane = tid % kWave, half = lane >> 5, l32 = lane & 31;
    const int ks = __builtin_amdgcn_readfirstlane(tid / kWave);

    // Logical tile -> output tile, in groups of 8 tile rows.
    const int width = 8 * tiles_n, grp = logical / width, first_m = grp * 8;
    const int gsize = tiles_m - first_m < 8 ? tiles_m - first_m : 8;
    const int64_t m0 = (int64_t)(first_m + (logical % width) % gsize) * BM, n0 = (int64_t)((logical % width) / gsize) * BN;

    // Two sums, as a sum rounds relative to its size.  fp32: the products of the first pieces by themselves, the other terms are small.
    // bf16 where the result is fp32: acc takes four steps (eight products), low all before them.  (As one sum a weight gradient over
    // K = 1000 / 2000 / 4000 was 1.9e-7 / 2.7e-7 / 3.9e-7 off on one wave, in fp32 products 0.9e-7 / 1.2e-7 / 1.7e-7, in two 0.8e-7 /
    // 1.0e-7 / 1.2e-7.  A bf16 result rounds by 2e-3: one sum is enough there, and leaves two waves their registers.)
    floatx16 acc[TM][TN], low[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = low[i][j][r] = 0.f;

    OA oa;
    OB ob;
    oa.init(a, lda, m0, M, lane);
    ob.init(b, ldb, n0, N, lane);
    char* ring = reinterpret_cast<char*>(red) + ks * 2 * STAGE;   // this wave's two stages
    typename OA::Raw ra[2];
    typename OB::Raw rb[2];
    GcFrag<T> fa[2][GROUPS][TM], fb[2][GROUPS][TN];
    uint32_t lost = 0;
    const int64_t steps = (K + KST - 1) / KST, mine = steps > ks ? (steps - ks + KS - 1) / KS : 0;   // this wave's: ks, ks + KS, ...
    // Whole steps: no piece of them reaches past the end of its operand (a piece of a ragged k-row may run into the rows after it).
    const int64_t over_a = AK || M % OA::EPP == 0 ? 0 : (OA::EPP - 2 + M) / M, over_b = BK || N % OB::EPP == 0 ? 0 : (OB::EPP - 2 + N) / N;
    const int64_t over = over_a > over_b ? over_a : over_b;
    const int64_t whole = K > over ? (K - over) / KST : 0, full = whole > ks ? (whole - ks + KS - 1) / KS : 0;
    auto load = [&](auto set, int64_t t) {
      constexpr int S = decltype(set)::v;
      const int64_t k = (t * KS + ks) * KST;
      if (t < full) {
        oa.load(ra[S], k);
        ob.load(rb[S], k);
      } else if (t < mine) {
        oa.template load_last<(KS > 1)>(ra[S], k, K, m0, M, lane);
        ob.template load_last<(KS > 1)>(rb[S], k, K, n0, N, lane);
      }
    };
    auto put = [&](auto set) {
      constexpr int S = decltype(set)::v;
      oa.put(ra[S], ring + S * STAGE, lane);
      ob.put(rb[S], ring + S * STAGE + OA::BYTES, lane);
    };
    auto cut = [&](auto set) {   // a step in LDS becomes operands
      constexpr int S = decltype(set)::v;
#pragma unroll
      for (int c = 0; c < GROUPS; ++c) {
        typename OA::Group ga;
        typename OB::Group gb;
        oa.get(ga, ring + S * STAGE, c, lane);
        ob.get(gb, ring + S * STAGE + OA::BYTES, c, lane);
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[S][c][i] = gc_cut(ga.v[i], lost);
#pragma unroll
        for (int j = 0; j < TN; ++j) fb[S][c][j] = gc_cut(gb.v[j], lost);
      }
    };
    auto products = [&](auto set) {
      constexpr int S = decltype(set)::v;
#pragma unroll
      for (int c = 0; c < GROUPS; ++c)
#pragma unroll
        for (int s = NP - 1; s >= 0; --s)   // pieces p + q = s
#pragma unroll
          for (int p = 0; p <= s; ++p)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
              for (int j = 0; j < TN; ++j) {
                floatx16& d = s ? low[i][j] : acc[i][j];
                d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[S][c][i].p[p], fb[S][c][j].p[s - p], d, 0, 0, 0);
              }
    };
    // Phase t: the products of step t, the cutting of step t + 1, step t + 2 into LDS, the loads of step t + 4.
    auto phase = [&](auto set, int64_t t, auto fast) {
      constexpr int S = decltype(set)::v;
      if constexpr (decltype(fast)::v) {
        put(set);
        oa.load(ra[S], ((t + 4) * KS + ks) * KST);
        ob.load(rb[S], ((t + 4) * KS + ks) * KST);
      } else {
        if (t + 2 < mine) put(set);
        load(set, t + 4);
      }
      gc_wave_order();   // (and left alone, the compiler sinks the loads to where they are needed)
      if constexpr (PARTS && S == 0) {
        if ((t & 2) == 0 || mine <= 16)   // (a short reduction: every two steps)
#pragma unroll
          for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
              low[i][j] += acc[i][j];
#pragma unroll
              for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
            }
      }
      if (decltype(fast)::v || t + 1 < mine) cut(GcInt<1 - S>{});
      products(set);
      if constexpr (NP > 1 && decltype(fast)::v) {
        __builtin_amdgcn_sched_group_barrier(0x100, 64, 0);
#pragma unroll
        for (int i = 0; i < 6 * TM * TN; ++i) {   // one product, then what issues in its shadow
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x002, TM * TN > 1 ? 9 : 16, 0);
        }
      }
      gc_wave_order();
    };
    int64_t t = 0;
    if (full > 5) {   // (no branch between here and the loop: at a join the compiler waits for every load)
      auto fetch = [&](auto set, int64_t u) {
        oa.load(ra[decltype(set)::v], (u * KS + ks) * KST);
        ob.load(rb[decltype(set)::v], (u * KS + ks) * KST);
        __builtin_amdgcn_sched_barrier(0);
      };
      fetch(GcInt<0>{}, 0);
      fetch(GcInt<1>{}, 1);
      put(GcInt<0>{});
      fetch(GcInt<0>{}, 2);
      put(GcInt<1>{});
      fetch(GcInt<1>{}, 3);
      gc_wave_order();
      cut(GcInt<0>{});
      do {
        phase(GcInt<0>{}, t, GcInt<1>{});
        phase(GcInt<1>{}, t + 1, GcInt<1>{});
        t += 2;
      } while (t + 5 < full);
    } else if (mine > 0) {
      load(GcInt<0>{}, 0);
      load(GcInt<1>{}, 1);
      put(GcInt<0>{});
      load(GcInt<0>{}, 2);
      if (mine > 1) put(GcInt<1>{});
      load(GcInt<1>{}, 3);
      gc_wave_order();
      cut(GcInt<0>{});
    }
    for (; t < mine; t += 2) {
      phase(GcInt<0>{}, t, GcInt<0>{});
      if (t + 1 < mine) phase(GcInt<1>{}, t + 1, GcInt<0>{});
    }

    if constexpr (NP > 1 || PARTS) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] += low[i][j];
    }
    if constexpr (NP > 1) {
      uint32_t mx = 0, mn = ~0u;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const uint32_t v = __builtin_bit_cast(uint32_t, (float)acc[i][j][r]) & 0x7fffffffu;
            mx = v > mx ? v : mx;
            mn = v - 1 < mn ? v - 1 : mn;   // (a sum of zero does not count)
          }
      // something is not finite, an operand had more bits than its pieces, or a sum is below 2^-100
      const bool inexact = __ballot(mx >= 0x7f800000u || (lost & 0xffffu) != 0 || mn < (27u << 23)) != 0;
      if (__builtin_expect(inexact, 0)) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            const int64_t m = m0 + OA::row(i, l32), n = n0 + OB::row(j, l32);
            const int64_t mr = m < M ? m : M - 1, nr = n < N ? n : N - 1;
            static_assert(KST == 16, "the steps of gc_exact_block");
            acc[i][j] = gc_exact_block<AK, BK>(a + mr * (AK ? lda : 1), b + nr * (BK ? ldb : 1), lda, ldb, K, ks, KS);
          }
      }
    }

    // acc[i][j][r] is row 8*(r/4) + 4*half + r%4, column l32 of its 32x32 block.
    auto row_of = [&](int i, int r) { return m0 + OA::row(i, 8 * (r >> 2) + 4 * half + (r & 3)); };
    auto fetch_old = [&](int i, int j, int r) {   // (past the end the last row or column)
      const int64_t m = row_of(i, r), n = n0 + OB::row(j, l32);
      return epilogue_fetch<T, MODE>(epi, m < M ? m : M - 1, n < N ? n : N - 1);
    };
    float bias[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int64_t n = n0 + OB::row(j, l32);
      bias[j] = epilogue_bias<T, MODE>(epi, n < N ? n : N - 1);
    }
    auto emit = [&](int i, int j, int r, float v, float old) {
      const int64_t m = row_of(i, r), n = n0 + OB::row(j, l32);
      if (m < M && n < N) epilogue_store<T, MODE>(epi, m, n, v, bias[j], old);
    };
    if constexpr (KS == 1) {
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        float old[16][TN];
#pragma unroll
        for (int r = 0; r < 16; ++r)
#pragma unroll
          for (int j = 0; j < TN; ++j) old[r][j] = fetch_old(i, j, r);
#pragma unroll
        for (int r = 0; r < 16; ++r)
#pragma unroll
          for (int j = 0; j < TN; ++j) emit(i, j, r, acc[i][j][r], old[r][j]);
      }
    } else {
      constexpr int RPW = 16 / KS;   // every wave finishes its share of the rows
      float old[TM][RPW][TN];
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int q = 0; q < RPW; ++q)
#pragma unroll
          for (int j = 0; j < TN; ++j) old[i][q][j] = fetch_old(i, j, ks * RPW + q);
      __syncthreads();   // (the sums lie where the waves' stages were)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) red[((ks * TM * TN + i * TN + j) * 16 + r) * 64 + lane] = acc[i][j][r];
      __syncthreads();
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int q = 0; q < RPW; ++q)
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            const int r = ks * RPW + q;
            float v = 0.f;
#pragma unroll
            for (int w = 0; w < KS; ++w) v += red[((w * TM * TN + i * TN + j) * 16 + r) * 64 + lane];
            emit(i, j, r, v, old[i][q][j]);
          }
    }
  }
};

// Workgroup -> tile: consecutive workgroups go round the 8 XCDs; every XCD gets a contiguous range of tiles, walked in
// groups of 8 tile rows (the panels it touches stay in its L2).
template <typename T, int MODE, bool AK, bool BK, int TM, int TN, int KS>
__global__ __launch_bounds__(KS * kWave) void gemm_cut_kernel(const T* __restrict__ a, int64_t lda, const T* __restrict__ b, int64_t ldb,
                                                              int64_t M, int64_t N, int64_t K, int tiles_m, int tiles_n, EpiArgs<T> epi) {
  extern __shared__ __attribute__((aligned(16))) float gc_smem[];
  int logical = blockIdx.x;
  const int nblk = gridDim.x;
  if ((nblk & 7) == 0) logical = (blockIdx.x & 7) * (nblk >> 3) + (blockIdx.x >> 3);
  if (gridDim.y > 1) {   // more than 2^22 tiles
    const int64_t t = (int64_t)blockIdx.y * nblk + logical;
    if (t >= (int64_t)tiles_m * tiles_n) return;
    logical = (int)t;
  }
  GcTile<T, MODE, AK, BK, TM, TN, KS>::run(a, lda, b, ldb, M, N, K, tiles_m, tiles_n, epi, logical, gc_smem);
}

// The jobs of gemm_f32_group_kernel.
template <typename T, int TM, int TN, int KS>
__global__ __launch_bounds__(KS * kWave) void gemm_cut_group_kernel(GfGroup<T> g) {
  extern __shared__ __attribute__((aligned(16))) float gc_smem[];
  using G = GcTile<T, EPI_ACCUM_F32, false, false, TM, TN, KS>;
  int j = 0;
  while (j + 1 < g.n && (int)blockIdx.x >= g.first[j + 1]) ++j;
  const WgradJob<T>& w = g.job[j];
  const int local = (int)blockIdx.x - g.first[j], nblk = g.first[j + 1] - g.first[j];
  const int logical = (local & 7) * (nblk >> 3) + (local >> 3);
  const int tiles_m = (w.M + G::BM - 1) / G::BM, tiles_n = (w.N + G::BN - 1) / G::BN;
  if (logical >= tiles_m * tiles_n) return;
  const EpiArgs<T> epi{nullptr, nullptr, nullptr, nullptr, w.out, w.N, DropArgs{}, 0};
  G::run(w.a, w.M, w.b, w.N, w.M, w.N, g.K, tiles_m, tiles_n, epi, logical, gc_smem);
}

// Which kernel a product takes: tile of 32 or 64 rows and columns and the number of waves that share it, or the fp32 products of gemm_f32.h.
//   bf16: as many waves as keep the chip's 1024 SIMDs busy.  Measured (us, 32x32 on 8 waves / 32x32 on 4 / 64x64 on 4 / 64x64 on 1):
//   301^3 4.6 / 5.3 / 9.2 / 16, [2001,131] over 601 7.5 / 7.5 / 10 / 18, [701,701] over 6001 50 / 46 / 47 / 59, 1001^3 18 / 17 / 15 / 22,
//   [4001,3001] over 3001 562 / 643 / 318 / 275.
//   Four waves on a tile also end each round with their sums' way through LDS, which a reduction of up to 256 does not pay for beyond one
//   round, of 256 tiles, or 512 in forward, whose workgroups share a CU (64x64 on 4 / on 1, forward, dgrad, wgrad): bf16 1550x1273 (500)
//   over 33 6.9 / 7.2, 12 / 7.6, 16 / 11 and over 200 7.9 / 9.1, 13 / 10, 18 / 18, 1803x1301 (609) over 104 11 / 8.9, 17 / 9.6, 23 / 15 and over 256
//   11 / 8.9, 21 / 13, 27 / 21; fp32 1803x1301 over 129 27 / 19, 27 / 17, 29 / 19 (fp32 products 25, 22, 26) and over 200 as dgrad 30 / 19, 1201x1101 (342) over 255 21 / 22, 21 / 20, 23 / 22.
//   (On fewer tiles a bf16 weight gradient over fewer than 64 tokens was 0.2 to 1.4 us shorter in fp32 products: 301x303 over 33 5.0 / 5.3,
//   701x1001 over 49 7.6 / 8.8.)
//   fp32 rows that are not whole 16-byte pieces, by the same rule from K = 128 on (fp32 products load such operands element by element; us,
//   those / this, forward, dgrad, wgrad): 301x303 over 301 8.4 / 5.2, 7.8 / 5.6, 8.3 / 6.3, 513x515 over 301 13.0 / 7.5, 11.2 / 7.7, 11.1 / 8.2,
//   1001x1003 over 201 13.8 / 11.3, 12.4 / 11.4, 16.9 / 12.5 and over 1003 39 / 24, 39 / 22, 47 / 23, 3001x3003 over 129 63 / 52, 56 / 46, 63 / 56;
//   but 3001x3003 over 33 28 / 45, 25 / 30, 36 / 68, 1729x355 over 65 7.4 / 8.6, 6.8 / 8.3, 7.6 / 11.7, 301x303 over 97 4.6 / 4.5, 4.6 / 4.9, 5.0 / 5.7.
//   fp32 in whole pieces (32x32 on 8 waves / 64x64 on 4 / 64x64 on 1 / fp32 products) from K = 1024 on: one round of 32x32 tiles, [512,512] over
//   2048 16 / 32 / 89 / 19 and 300x300 over 1200 11 / 22 / 58 / 12.5; from two thirds of a round of 64x64 tiles, 1024^3 38 / 24 / 54 / 30,
//   1500^3 137 / 87 / 90 / 98, 2048^3 235 / 167 / 147 / 184.  64x64 on 4 waves come in whole rounds of 256, so they pay where the fp32
//   products' own rounds (gf_small_tile, there on 32x32 tiles four times finer) take 3.5 times the tile area per round, 4 times
//   below K = 1280 (fp32 products / 64x64 on 4, forward, dgrad, wgrad): at 3 times, 500x2304 over 1024 33 / 40, 32 / 38, 35 / 43 and over 2048
//   60 / 65, 58 / 63, 63 / 69; at 3.6, 1024x2304 over 1024 59 / 61, 58 / 58, 60 / 66, over 1280 73 / 72, 72 / 69, 75 / 76 and over 2048
//   114 / 101, 109 / 98, 111 / 105; at 4, 1000x1600 over 1024 42 / 40, 42 / 38, 47 / 44.  A shorter reduction does not pay for the sums' way through LDS:
//   [1000,768] over 768 26 / 20 / 43 / 20, transposed operands 29 / 24 / 54 / 20, 256x256 over 512 6.2 / 13 / 31 / 6.6, transposed
//   7.0 / 15 / 34 / 6.8, 128x512 over 128 4.2 / 8.2 / 17 / 3.8.
enum GcKind : int { GC_NONE = 0, GC_32_8 = 1, GC_32_4 = 2, GC_64_4 = 3, GC_64_1 = 4 };
inline GcKind gc_kind(bool fp32, bool pieces, bool forward, int64_t tiles32, int64_t tiles64, int64_t K) {
  if (fp32 && K < (pieces ? 1024 : 128)) return GC_NONE;
  if (tiles32 <= 256) return GC_32_8;
  if (!fp32 || !pieces) return tiles32 <= 512 ? GC_32_4 : tiles64 <= (K > 256 ? 768 : forward ? 512 : 256) ? GC_64_4 : GC_64_1;
  if (tiles64 >= 768) return GC_64_1;
  const double r32 = (double)((tiles32 + 255) / 256), r64 = (double)((tiles64 + 255) / 256);
  const double area = gf_small_tile(tiles32, tiles64) ? 1.2 * r32 : 4.0 * r64;
  return tiles64 >= 170 && area >= (K < 1280 ? 4.0 : 3.5) * r64 ? GC_64_4 : GC_NONE;
}

}  // namespace varuna
