// GEMM with fp32 products and fp32 accumulation on the matrix cores (v_mfma_f32_32x32x2_f32):
//   acc[m,n] = sum_k A(m,k) * B(n,k)
//   AK: A(m,k) = a[m*lda + k]   else A(m,k) = a[k*lda + m];   BK likewise for B(n,k) = b[n*ldb + k] / b[k*ldb + n]
// It serves the fp32 path where products of bf16 pieces (gemm_cut.h) are no faster: short reductions, below K = 1024 over whole 16-byte
// pieces and below 128 over others (gc_kind).  Any M, N, K; every global access is bounds-checked.
//
// What bounds it: the fp32 matrix rate, 256 FLOP per clock and CU (157 TFLOP/s nominal, the rate a large library
// product reaches here); a product of a 32x32 block takes 64 clocks for two LDS words per lane, so neither LDS
// nor issue is close.  At the sizes of the fp32 path (a few hundred to a thousand tokens) what counts instead is
// filling 1024 SIMDs: KS waves of a workgroup share an output tile and take every stage's k-range in KS parts,
// summed through LDS in a fixed order at the end, so a 32x32 tile still occupies all four SIMDs of its CU, and
// stages are long (64 or 128 k), which leaves a load's latency the products of the resident workgroups.  Measured
// against the vector-ALU kernel before it (us): [128,128] over 512 60 -> 5; [1000,768] over 768 takes 20, and 2048^3 ran at 111 TFLOP/s.
#pragma once
#include "common.h"
#include "gemm_epilogue.h"

namespace varuna {

// LDS tile of ROWS x BKT floats.  KMAJOR: [row][BKT + 4] (an odd number of 16-byte pieces per row: 16-byte reads of
// consecutive rows fall into different banks); else [k][ROWS + 8] (k-rows four apart, the distance between the two
// half waves of a read, are half of the banks apart).
template <int ROWS, int BKT, bool KMAJOR>
struct GfTile {
  static constexpr int PITCH = KMAJOR ? BKT + 4 : ROWS + 8;
  static constexpr int ELEMS = KMAJOR ? ROWS * PITCH : BKT * PITCH;
};

// Staging of one operand tile: global -> registers -> LDS, four consecutive elements of the contiguous direction
// at a time.  VEC: one 16-byte load per piece, which needs an aligned base, a leading dimension and a contiguous extent that are
// multiples of 4; otherwise element by element.  Outside the matrix: zeros.
template <int ROWS, int BKT, bool KMAJOR, bool VEC, int NT>
struct GfLoader {
  static constexpr int PIECES = ROWS * BKT / 4, PPT = PIECES / NT;
  static_assert(PIECES % NT == 0, "tile / threads mismatch");
  floatx4 v[PPT];
  __device__ __forceinline__ void load(const float* __restrict__ g, int64_t ld, int64_t row0, int64_t rows, int64_t k0, int64_t K, int tid) {
#pragma unroll
    for (int i = 0; i < PPT; ++i) {
      const int id = tid + i * NT;
      constexpr int PPL = (KMAJOR ? BKT : ROWS) / 4;   // pieces per line of the contiguous direction
      const int line = id / PPL, c = (id % PPL) * 4;
      const int64_t row = row0 + (KMAJOR ? line : c), k = k0 + (KMAJOR ? c : line);
      const bool line_ok = KMAJOR ? row < rows : k < K;
      const int64_t left = KMAJOR ? K - k : rows - row;   // elements of the contiguous direction from here on
      const float* p = g + (KMAJOR ? row * ld + k : k * ld + row);
      floatx4 x = {0.f, 0.f, 0.f, 0.f};
      if constexpr (VEC) {
        if (line_ok && left > 0) x = *reinterpret_cast<const floatx4*>(p);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (line_ok && left > e) x[e] = p[e];
      }
      v[i] = x;
    }
  }
  __device__ __forceinline__ void store(float* __restrict__ lds, int tid) const {
#pragma unroll
    for (int i = 0; i < PPT; ++i) {
      const int id = tid + i * NT;
      constexpr int PPL = (KMAJOR ? BKT : ROWS) / 4;
      *reinterpret_cast<floatx4*>(lds + (id / PPL) * GfTile<ROWS, BKT, KMAJOR>::PITCH + (id % PPL) * 4) = v[i];
    }
  }
};

// Four products' worth of one operand: element i of the result belongs to product i, whose two k-values are
// kg + i (lower half wave) and kg + 4 + i (upper half wave).
template <int ROWS, int BKT, bool KMAJOR>
__device__ __forceinline__ floatx4 gf_frag(const float* lds, int row, int kg, int half) {
  constexpr int P = GfTile<ROWS, BKT, KMAJOR>::PITCH;
  if constexpr (KMAJOR) return *reinterpret_cast<const floatx4*>(lds + row * P + kg + 4 * half);
  const float* p = lds + (kg + 4 * half) * P + row;
  return floatx4{p[0], p[P], p[2 * P], p[3 * P]};
}

// One workgroup: a BM x BN tile on (BM / WM) * (BN / WN) * KS waves, one stage of BKT k in LDS, the next in registers.
template <int MODE, bool AK, bool BK, int BM, int BN, int WM, int WN, int KS, int BKT, bool VEC>
__device__ __forceinline__ void gf_tile(
    const float* __restrict__ a, int64_t lda, const float* __restrict__ b, int64_t ldb, int64_t M, int64_t N, int64_t K,
    int tiles_m, int tiles_n, const EpiArgs<float>& epi, int logical) {
  constexpr int NW = (BM / WM) * (BN / WN) * KS, NT = NW * kWave;
  constexpr int TM = WM / 32, TN = WN / 32;
  constexpr int AE = GfTile<BM, BKT, AK>::ELEMS, BE = GfTile<BN, BKT, BK>::ELEMS;
  constexpr int STAGE = AE + BE;
  constexpr int RED = KS > 1 ? NW * TM * TN * 1024 : 0;   // floats of the partial sums
  __shared__ __attribute__((aligned(16))) float smem[STAGE > RED ? STAGE : RED];
  const int tid = threadIdx.x, lane = tid % kWave, half = lane >> 5, l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int ks = wave % KS, wt = wave / KS, wm = wt / (BN / WN), wn = wt % (BN / WN);

  // Logical tile -> output tile, in groups of 8 tile rows.
  const int width = 8 * tiles_n, grp = logical / width, first_m = grp * 8;
  const int gsize = tiles_m - first_m < 8 ? tiles_m - first_m : 8;
  const int64_t m0 = (int64_t)(first_m + (logical % width) % gsize) * BM, n0 = (int64_t)((logical % width) / gsize) * BN;

  floatx16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  GfLoader<BM, BKT, AK, VEC, NT> la;
  GfLoader<BN, BKT, BK, VEC, NT> lb;
  const int64_t nst = (K + BKT - 1) / BKT;
  la.load(a, lda, m0, M, 0, K, tid);
  lb.load(b, ldb, n0, N, 0, K, tid);
  la.store(smem, tid);
  lb.store(smem + AE, tid);
  __syncthreads();
  const float* sa = smem;
  const float* sb = smem + AE;
  for (int64_t st = 0; st < nst; ++st) {
    if (st + 1 < nst) {   // in flight during this stage's products
      la.load(a, lda, m0, M, (st + 1) * BKT, K, tid);
      lb.load(b, ldb, n0, N, (st + 1) * BKT, K, tid);
    }
    constexpr int GROUPS = BKT / (8 * KS);
#pragma unroll
    for (int g = 0; g < GROUPS; ++g) {
      const int kg = (ks * GROUPS + g) * 8;
      floatx4 fa[TM], fb[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) fa[i] = gf_frag<BM, BKT, AK>(sa, wm * WM + i * 32 + l32, kg, half);
#pragma unroll
      for (int j = 0; j < TN; ++j) fb[j] = gf_frag<BN, BKT, BK>(sb, wn * WN + j * 32 + l32, kg, half);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i][e], fb[j][e], acc[i][j], 0, 0, 0);
    }
    if (st + 1 < nst) {
      __syncthreads();
      la.store(smem, tid);
      lb.store(smem + AE, tid);
      __syncthreads();
    }
  }

  // acc[i][j][r] is row 8*(r/4) + 4*half + r%4, column l32 of its 32x32 block.
  const int64_t mb = m0 + wm * WM, nb = n0 + wn * WN;
  auto put = [&](int i, int j, int r, float v) {
    const int64_t m = mb + i * 32 + 8 * (r >> 2) + 4 * half + (r & 3), n = nb + j * 32 + l32;
    if (m < M && n < N) epilogue_store<float, MODE>(epi, m, n, v);
  };
  if constexpr (KS == 1) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) put(i, j, r, acc[i][j][r]);
  } else {
    __syncthreads();   // the stages are read no more
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) smem[((wave * TM * TN + i * TN + j) * 16 + r) * 64 + lane] = acc[i][j][r];
    __syncthreads();
    constexpr int RPW = 16 / KS;   // every wave finishes its share of the rows
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int q = 0; q < RPW; ++q) {
          const int r = ks * RPW + q;
          float v = 0.f;
#pragma unroll
          for (int p = 0; p < KS; ++p) v += smem[(((wt * KS + p) * TM * TN + i * TN + j) * 16 + r) * 64 + lane];
          put(i, j, r, v);
        }
  }
}

// Workgroup -> tile: consecutive workgroups go round the 8 XCDs; every XCD gets a contiguous range of tiles, walked in
// groups of 8 tile rows (the panels it touches stay in its L2).
template <int MODE, bool AK, bool BK, int BM, int BN, int WM, int WN, int KS, int BKT, bool VEC>
__global__ __launch_bounds__((BM / WM) * (BN / WN) * KS * kWave) void gemm_f32_kernel(
    const float* __restrict__ a, int64_t lda, const float* __restrict__ b, int64_t ldb, int64_t M, int64_t N, int64_t K,
    int tiles_m, int tiles_n, EpiArgs<float> epi) {
  int logical = blockIdx.x;
  const int nblk = gridDim.x;
  if ((nblk & 7) == 0) logical = (blockIdx.x & 7) * (nblk >> 3) + (blockIdx.x >> 3);
  if (gridDim.y > 1) {   // more than 2^22 tiles
    const int64_t t = (int64_t)blockIdx.y * nblk + logical;
    if (t >= (int64_t)tiles_m * tiles_n) return;
    logical = (int)t;
  }
  gf_tile<MODE, AK, BK, BM, BN, WM, WN, KS, BKT, VEC>(a, lda, b, ldb, M, N, K, tiles_m, tiles_n, epi, logical);
}

// A layer norm in front of a product (gemm_f32_few.h): parameters, and where the normalised rows, the statistics (mean, then reciprocal standard
// deviation) and a copy of the rows go (each may be null).
struct LnIn {
  const float *gamma, *beta;
  float *y, *stats, *copy;
  float eps;
};

// Several weight gradients out[M,N] += a[K,M]^T b[K,N] over the same K in one launch: the products of a small stage are a few
// microseconds each, less than what lies between two launches, and those of a larger one each end with a partly filled
// round.  Job j owns workgroups first[j] .. first[j+1]-1, a multiple of 8 of them; those past its last tile end at once.
template <typename T>
struct GfGroup {
  int n;
  int64_t K;
  int first[kMaxGroupJobs + 1];
  WgradJob<T> job[kMaxGroupJobs];
};
template <int BM, int BN, int WM, int WN, int KS, int BKT, bool VEC>
__global__ __launch_bounds__((BM / WM) * (BN / WN) * KS * kWave) void gemm_f32_group_kernel(GfGroup<float> g) {
  int j = 0;
  while (j + 1 < g.n && (int)blockIdx.x >= g.first[j + 1]) ++j;
  const WgradJob<float>& w = g.job[j];
  const int local = (int)blockIdx.x - g.first[j], nblk = g.first[j + 1] - g.first[j];
  const int logical = (local & 7) * (nblk >> 3) + (local >> 3);
  const int tiles_m = (w.M + BM - 1) / BM, tiles_n = (w.N + BN - 1) / BN;
  if (logical >= tiles_m * tiles_n) return;
  const EpiArgs<float> epi{nullptr, nullptr, nullptr, nullptr, w.out, w.N, DropArgs{}, 0};
  gf_tile<EPI_ACCUM_F32, false, false, BM, BN, WM, WN, KS, BKT, VEC>(w.a, w.M, w.b, w.N, w.M, w.N, g.K, tiles_m, tiles_n, epi, logical);
}

// Output tile of a product: 64x64 (4 waves of 32x32) or 32x32 (8 waves, each an eighth of every stage's k-range).
// Either occupies the four SIMDs of a CU, so a product takes about ceil(tiles / 256) times the tile's area, and the
// small tile loses 1.2x to its larger traffic per product.  Measured (us, 64x64 / 32x32): 1000x768x3072 75 / 62,
// 768x768x1000 27 / 22, 1000x3072x768 53 / 64, 2048x2048x2048 155 / 188; 128x128x512 15.6 / 9.4 with the launch.
// (128x128 tiles: 152 at 2048^3, 220 and more at the others.)
inline int64_t gf_tiles(int64_t M, int64_t N, int64_t size) { return ((M + size - 1) / size) * ((N + size - 1) / size); }
inline bool gf_small_tile(int64_t tiles32, int64_t tiles64) {
  return 1.2 * (double)((tiles32 + 255) / 256) * (32 * 32) < (double)((tiles64 + 255) / 256) * (64 * 64);
}

// Products of few output elements, or of short sums, go to gemm_f32_few.h (forward and dgrad, whole 16-byte pieces), in
// 16x16 tiles.  Measured (us, tiles of 32 or 64 / that, forward and dgrad): 128x128 (64 tiles) over 128 3.6 / 2.4, 3.6 / 2.3 and over 512
// 6.2 / 3.7, 6.2 / 3.2, 128x512 (256) over 900 9.9 / 4.3, 9.8 / 4.3, 256x512 (512) over 512 6.3 / 5.6, 6.4 / 4.7 and over 1000
// 9.9 / 7.0, 9.8 / 6.9, 512x512 (1024) over 64 3.7 / 3.2, 3.8 / 3.0 and over 128 3.8 / 3.9, 3.9 / 3.4, 2000x256 (2000) over 64 4.9 / 4.5,
// 4.8 / 4.2; beyond, 256x768 (768) over 256 4.6 / 4.7, 4.7 / 4.0, 500x384 (768) over 384 5.6 / 6.4, 5.5 / 5.4, 512x512 over 512 6.5 / 9.1, 6.5 / 6.8.
// From 1024 k on the kernels on bf16 pieces take products this small (gc_kind); these take two batches of 512 k and address an operand (at
// most 32768 rows of it) with 32 bits.
inline bool gf_few(int64_t M, int64_t N, int64_t K) {
  const int64_t tiles = gf_tiles(M, N, 16);
  return K < 1024 && (tiles <= 512 || (tiles <= 2048 && tiles * K <= 1 << 17));
}

// One product on contiguous operands (forward: a [M,K], b [N,K]; dgrad: [M,K], [K,N]; wgrad: [K,M], [K,N]), in
// gemm_f32.hip (T = float) and gemm_f32_bf16.hip.
template <typename T>
hipError_t launch_gemm_f32(int op, int mode, const T* a, const T* b, int64_t M, int64_t N, int64_t K, const EpiArgs<T>& epi,
                           hipStream_t st);

// The same product in front of which a layer norm of a's rows stands (EPI_BIAS and EPI_BIAS_GELU), in one launch, where it takes the shape and the
// tensors (ln_gemm_f32_takes).  A norm on its own is a launch of 3 us, most of it latency: steps of two layers 128 wide, four micro-batches of 128 tokens, 668 -> 598 us.
bool ln_gemm_f32_takes(const float* b, const LnIn& ln, int64_t M, int64_t N, int64_t K);
hipError_t launch_ln_gemm_f32(int mode, const float* a, const float* b, int64_t M, int64_t N, int64_t K, const EpiArgs<float>& epi, const LnIn& ln, hipStream_t st);

// `n` weight gradients over K (all of a layer, of several layers), in one launch of gemm_f32.hip.  One by one against one launch:
// two layers 128 wide over 128 tokens 8 x 3.9 against 6.5 us, one layer 768 wide over 1000 tokens 206 against 164 us.
hipError_t launch_gemm_f32_group(const WgradJob<float>* jobs, int n, int64_t K, hipStream_t st);
// The same on bf16 operands (products of gemm_cut.h), in gemm_f32_bf16.hip.
hipError_t launch_gemm_cut_group(const WgradJob<bf16>* jobs, int n, int64_t K, hipStream_t st);

}  // namespace varuna
