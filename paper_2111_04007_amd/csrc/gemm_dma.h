// bf16 MFMA GEMM for gfx950: operands go from global memory straight into LDS
// (buffer_load_dwordx4 ... lds, no register staging) into stages of 64 k (two per
// operand, two of A and three of B, or three of both: template parameter LS), and MFMA fragments
// are software-pipelined in registers across k-steps and across k-tiles, with one
// workgroup barrier per k-tile.
//
//   acc[m,n] = sum_k A(m,k) * B(n,k)
//   A_KMAJOR: A(m,k) = a[m*lda + k]   else (m-major): A(m,k) = a[k*lda + m]
//   B_KMAJOR: B(n,k) = b[n*ldb + k]   else (n-major): B(n,k) = b[k*ldb + n]
//
// LDS layouts (each wave-level direct load deposits 64 lanes x 16 B contiguously,
// so swizzles are applied by choosing which global chunk a lane fetches):
//   k-major operand : [row][64 k]  (128 B per row, 8 chunks of 16 B),
//                     physical chunk = c ^ ((row ^ (row >> 3)) & 7); fragments by ds_read_b128.
//   m/n-major operand: [k][ROWS]   (ROWS*2 B per k-row), physical chunk within each
//                     group of 16 = c ^ dg_tr_swizzle(k); fragments by the transposing
//                     LDS read ds_read_b64_tr_b16 (16 lanes x 4 k-rows -> each lane
//                     gets 4 consecutive k of its own row), two per 8-k operand.
// Both give a lane the 8 consecutive k-values (lane/32)*8.. of tile row lane%32,
// which is the operand layout of v_mfma_f32_32x32x16_bf16.
#pragma once
#include <type_traits>

#include "common.h"
#include "gemm_epilogue.h"

namespace varuna {

constexpr int DG_BK = 64;      // k per LDS stage: 128-byte row segments keep the L1/L2 path efficient
constexpr int DG_STAGES = 2;

typedef short shortx4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void* lds_ptr_t;
typedef const __attribute__((address_space(1))) void* glb_ptr_t;

// s_waitcnt immediates (gfx9 encoding: vmcnt [3:0]+[15:14], expcnt [6:4], lgkmcnt [11:8]).
#define DG_WAIT_VM(n) (((n) & 0xf) | (((n) >> 4) << 14) | (7 << 4) | (15 << 8))
#define DG_WAIT_VM0_LGKM0 (7 << 4)
#define DG_WAIT_LGKM0 (0xf | (3 << 14) | (7 << 4))

// Direct global->LDS staging of one operand tile (ROWS x 64).
//   k-major  : LDS [row][64 k], 8 chunks of 16 B per row, physical chunk = c ^ ((row ^ (row >> 3)) & 7)
//   m/n-major: LDS [k][ROWS],   physical chunk (within each aligned group of 16) = c ^ dg_tr_swizzle(k)
// A transposing read takes, per 16 lanes, 32 B from each of 4 consecutive k-rows, and per 32 lanes 64 B
// from each; k-rows are a multiple of 256 B apart, so unswizzled all four start in the same bank.  The
// XOR values 0, 6, 12, 10 differ both in bits 1-2 and in bits 2-3 of the chunk number: the four rows'
// 32-byte pieces fall into different quarters of 128 B and their 64-byte pieces into different quarters
// of 256 B, which is free of bank conflicts whether the LDS serves 16 or 32 lanes of such a read at once.
__device__ __forceinline__ constexpr int dg_tr_swizzle(int k) { return ((k & 1) * 6) ^ (((k >> 1) & 1) * 12); }

//
// EDGE: the operand's rows or its reduction may end inside the tile.  Rows past the end repeat the last one (k-major) or
// read the next k-row (m/n-major); they only reach outputs that are not stored.  k past the end must read as zero in
// both operands (a foreign value there could be a NaN): it lies past the buffer's extent (m/n-major), and in a k-major
// operand the last k-tile uses offsets that put every chunk past the end of its row outside the buffer.
// Only loads of the last k-tile can lie outside as a whole (see the wait before the barrier).
constexpr uint32_t DG_OUTSIDE = 0x80000000u;   // past the extent of any EDGE operand (below 2 GiB), whatever k-tile is added
template <int ROWS, int NW, bool KMAJOR, bool EDGE = false>
struct DgLoader {
  static constexpr int NINS = ROWS * DG_BK * 2 / 1024;  // wave-level 1 KB loads per tile
  static constexpr int LPT = NINS / NW;                  // per wave
  static_assert(NINS % NW == 0 && LPT >= 1, "tile rows / waves mismatch");
  static_assert(KMAJOR || ROWS % 128 == 0, "the m/n-major swizzle permutes groups of 16 chunks");
  const bf16* base;             // the whole operand is one buffer; loads beyond its extent return zero
  uint32_t extent;
  uint32_t voff[LPT];           // per-lane byte offset of each of this wave's loads (k-tile 0)
  uint32_t step;                // bytes to advance per k-tile
  uint32_t vtail[EDGE && KMAJOR ? LPT : 1];   // voff in the last k-tile
  int last_kt;

  // rows: of the whole operand; k_tail: k in the last k-tile (1..64), which has number last_tile
  __device__ __forceinline__ void init(const bf16* g, int64_t ld, int64_t row0, int wave, int lane, uint32_t extent_bytes,
                                       int64_t rows, int k_tail, int last_tile) {
    base = g;
    extent = extent_bytes;
    last_kt = last_tile;
#pragma unroll
    for (int i = 0; i < LPT; ++i) {
      const int q = wave + i * NW;
      if (KMAJOR) {
        const int row = q * 8 + (lane >> 3), p = lane & 7;
        const int c = p ^ ((row ^ (row >> 3)) & 7);
        const int64_t grow = EDGE && row0 + row >= rows ? rows - 1 : row0 + row;
        voff[i] = (uint32_t)((grow * ld + c * 8) * 2);
        if constexpr (EDGE) vtail[i] = c * 8 < k_tail ? voff[i] : DG_OUTSIDE;
      } else {
        constexpr int CPR = ROWS / 8;  // chunks per k-row
        const int slot = q * 64 + lane, krow = slot / CPR, p = slot % CPR;
        const int c = p ^ dg_tr_swizzle(krow);
        voff[i] = (uint32_t)(((int64_t)krow * ld + row0 + c * 8) * 2);
      }
    }
    step = (uint32_t)((KMAJOR ? (int64_t)DG_BK : (int64_t)DG_BK * ld) * 2);
  }

  __device__ __forceinline__ uint32_t offset(int i, int kt) const {
    if constexpr (EDGE && KMAJOR) return kt == last_kt ? vtail[i] : voff[i];
    return voff[i];
  }
  __device__ __forceinline__ void issue(bf16* lds_tile, int kt, int wave) const {
#if defined(__HIP_DEVICE_COMPILE__)  // the buffer builtins exist in the device pass only
    const uint32_t soff = (uint32_t)kt * step;
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16*>(base), 0, extent, 0x00020000);
#pragma unroll
    for (int i = 0; i < LPT; ++i) {
      const int q = wave + i * NW;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_ptr_t)(lds_tile + q * 512), 16, offset(i, kt), soff, 0, 0);
    }
#endif
  }
  // Load number I of this wave alone.  With live == false the descriptor covers zero bytes: every
  // lane is out of range, no memory request is made and the load only deposits zeros, so a
  // k-tile past the end of the reduction costs no branch in the middle of a run of products.
  template <int I>
  __device__ __forceinline__ void issue_one(bf16* lds_tile, int kt, int wave, bool live) const {
#if defined(__HIP_DEVICE_COMPILE__)
    static_assert(I >= 0 && I < LPT, "load index");
    const uint32_t soff = (uint32_t)kt * step;
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16*>(base), 0, live ? extent : 0u, 0x00020000);
    const int q = wave + I * NW;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_ptr_t)(lds_tile + q * 512), 16, offset(I, kt), live ? soff : 0u, 0, 0);
#endif
  }
};

// One MFMA operand fragment in registers.  In a kernel whose operands are both k-major the
// fragments are plain 16-byte LDS loads that the compiler tracks and schedules (HAND = false).
// A kernel with an m/n-major operand issues ALL its fragment reads as inline assembly
// (HAND = true): the compiler treats the transposing-read builtin as a possible alias of the
// direct-to-LDS loads and puts a wait for all of them (vmcnt(0)) in front of the first such
// read after every issue of the next k-tile, which exposes the full memory latency once per
// k-tile.  Reads it does not see cost no such wait; their completion is waited for by hand
// (settle() before the first use), and issue order is source order.
template <bool KMAJOR, bool HAND> struct DgFragReg;
template <> struct DgFragReg<true, false> { bf16x8 v; };
template <> struct DgFragReg<true, true> { bf16x8 v; };
template <> struct DgFragReg<false, true> { shortx4 lo, hi; };

template <bool HAND> __device__ __forceinline__ bf16x8 dg_value(const DgFragReg<true, HAND>& f) { return f.v; }
__device__ __forceinline__ bf16x8 dg_value(const DgFragReg<false, true>& f) {
  union { struct { shortx4 a, b; } s; bf16x8 v; } u;
  u.s.a = f.lo; u.s.b = f.hi;
  return u.v;
}
// Waits until every LDS read this wave has issued so far has returned; tied to the fragment's
// registers so that no use of them can be scheduled above it.
__device__ __forceinline__ void dg_settle(DgFragReg<true, false>&) {}
__device__ __forceinline__ void dg_settle(DgFragReg<true, true>& f) { asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(f.v)); }
__device__ __forceinline__ void dg_settle(DgFragReg<false, true>& f) {
  asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(f.lo), "+v"(f.hi));
}
// The same for a whole array of fragments with one wait.
template <int N> __device__ __forceinline__ void dg_settle_all(DgFragReg<true, false> (&)[N]) {}
template <int N> __device__ __forceinline__ void dg_settle_all(DgFragReg<true, true> (&f)[N]) {
  if constexpr (N == 2) asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(f[0].v), "+v"(f[1].v));
  else if constexpr (N == 4) asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(f[0].v), "+v"(f[1].v), "+v"(f[2].v), "+v"(f[3].v));
  else {
#pragma unroll
    for (int i = 0; i < N; ++i) dg_settle(f[i]);
  }
}
template <int N> __device__ __forceinline__ void dg_settle_all(DgFragReg<false, true> (&f)[N]) {
  if constexpr (N == 2) asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(f[0].lo), "+v"(f[0].hi), "+v"(f[1].lo), "+v"(f[1].hi));
  else if constexpr (N == 4)
    asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(f[0].lo), "+v"(f[0].hi), "+v"(f[1].lo), "+v"(f[1].hi), "+v"(f[2].lo), "+v"(f[2].hi),
                 "+v"(f[3].lo), "+v"(f[3].hi));
  else {
#pragma unroll
    for (int i = 0; i < N; ++i) dg_settle(f[i]);
  }
}

// Fragment reader: the 8 consecutive k-values KS*16 + (lane/32)*8 .. of row lane%32 of fragment number IDX
// (32 rows each) of the wave's sub-tile, whose first row is wave_base (a multiple of 32).  Fragment number
// and k-step are compile-time values: in the hand-issued forms whatever part of the address they contribute
// additively goes into the instruction's offset field instead of into an address computation.
template <int ROWS, bool KMAJOR, bool HAND>
struct DgFrag {
  template <int IDX, int KS>
  static __device__ __forceinline__ void fetch(DgFragReg<KMAJOR, HAND>& f, const bf16* lds_tile, int wave_base,
                                               std::integral_constant<int, IDX>, std::integral_constant<int, KS>, int lane) {
    if constexpr (KMAJOR) {
      // the swizzle depends on the fragment number through its parity only: row bits 3..5 are 4*IDX + lane bits
      const int row = wave_base + (IDX & 1) * 32 + (lane & 31), c = KS * 2 + (lane >> 5);
      const bf16* p0 = lds_tile + row * DG_BK + ((c ^ ((row ^ (row >> 3)) & 7)) << 3);
      constexpr int IMM = (IDX >> 1) * 64 * DG_BK * 2;   // bytes
      if constexpr (HAND) {
        const uint32_t a0 = (uint32_t)(uintptr_t)(lds_ptr_t)const_cast<bf16*>(p0);
        asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(f.v) : "v"(a0), "n"(IMM));
      } else {
        f.v = *reinterpret_cast<const bf16x8*>(reinterpret_cast<const unsigned char*>(p0) + IMM);
      }
    } else {
      const int blk = lane >> 4, j = lane & 15;
      const int m = wave_base + IDX * 32 + (blk & 1) * 16 + 4 * (j & 3);
      const int kq = j >> 2;  // k-row within its group of 4 == (krow & 3)
      const int c = m >> 3, phys = c ^ dg_tr_swizzle(kq);
      const bf16* p0 = lds_tile + ((blk >> 1) * 8 + kq) * ROWS + phys * 8 + (m & 7);
      const uint32_t a0 = (uint32_t)(uintptr_t)(lds_ptr_t)const_cast<bf16*>(p0);
      constexpr int IMM0 = KS * 16 * ROWS * 2, IMM1 = IMM0 + 4 * ROWS * 2;   // bytes
      static_assert(IMM1 < 65536, "offset field");
      asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(f.lo) : "v"(a0), "n"(IMM0));
      asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(f.hi) : "v"(a0), "n"(IMM1));
    }
  }
};

// Scheduling hints for one k-step: MFMA, then RPM LDS reads (and one direct load if any
// are pending in this step), MFMA, ...
template <int Q, int NMFMA, int NREAD, int RPM, int NVMEM>
struct DgInterleave {
  static __device__ __forceinline__ void hint() {
    if constexpr (Q < NMFMA) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      if constexpr (Q * RPM < NREAD)
        __builtin_amdgcn_sched_group_barrier(0x100, (Q * RPM + RPM <= NREAD) ? RPM : NREAD - Q * RPM, 0);
      if constexpr (Q < NVMEM) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
      DgInterleave<Q + 1, NMFMA, NREAD, RPM, NVMEM>::hint();
    }
  }
};

// f(integral_constant<int, 0>) ... f(integral_constant<int, N-1>), unrolled at compile time.
template <int N, typename F>
__device__ __forceinline__ void dg_static_for(F&& f) {
  if constexpr (N > 0) {
    dg_static_for<N - 1>(f);
    f(std::integral_constant<int, N - 1>{});
  }
}
// A half-open range of load numbers handed to one k-step.
template <int LO, int HI> struct DgLoads { static constexpr int lo = LO, hi = HI; };
// Load number J (LO <= J < HI) goes out right after product number dg_load_slot of the k-step's NMFMA.
constexpr int dg_load_slot(int j, int lo, int hi, int nmfma) { return ((j - lo) * nmfma) / (hi - lo); }
constexpr uint32_t dg_load_mask(int lo, int hi, int nmfma) {
  uint32_t m = 0;
  for (int j = lo; j < hi; ++j) m |= 1u << dg_load_slot(j, lo, hi, nmfma);
  return m;
}
// Scheduling hints for one k-step whose direct loads sit after the products named in VMASK.
template <int Q, int NMFMA, int NREAD, int RPM, uint32_t VMASK>
struct DgInterleaveMask {
  static __device__ __forceinline__ void hint() {
    if constexpr (Q < NMFMA) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      if constexpr (Q * RPM < NREAD)
        __builtin_amdgcn_sched_group_barrier(0x100, (Q * RPM + RPM <= NREAD) ? RPM : NREAD - Q * RPM, 0);
      if constexpr ((VMASK >> Q) & 1u) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
      DgInterleaveMask<Q + 1, NMFMA, NREAD, RPM, VMASK>::hint();
    }
  }
};

// bf16 epilogue of one wave's (TM*32) x WN sub-tile whose first output is (row0, col0), through a
// private LDS buffer of 32 rows x WN floats.  acc[i][j][r] is row m = lane%32 of the 32x32 block,
// column n = 8*(r/4) + 4*(lane/32) + r%4.  Columns WN of the sub-tile from block J0 on (32 or a multiple of 64 at a time).
// Bound by memory: what it reads of the output's shape (aux_in) goes out a pass ahead, and the bias once.  Read where they are used, each of the
// 16 or 32 row groups waited for a round trip, behind its predecessor's store.  Before / after (us, operands out of cache): residual
// 4096x7680x1920 153 / 116, 4096x4096x1024 63 / 44, 4096x1024x1024 17.3 / 14.0, 2000x1600x1600 22.1 / 18.8 (without the residual 102, 36, 13.1, 17.9);
// GeLU' 4096x7680x1920 135 / 121, 4096x1920x1920 46.6 / 38.3; bias alone 4096x12288x3072 247 / 236, 4096x3072x1024 32.8 / 28.6.
template <int MODE, int TM, int TN, int WN, bool EDGE, int J0 = 0>
__device__ __forceinline__ void dg_epilogue_bf16(floatx16 (&acc)[TM][TN], unsigned char* buf, const EpiArgs<bf16>& epi,
                                                 int64_t row0, int64_t col0, int lane, int64_t rows, int64_t cols) {
  constexpr int ROWB = WN * 4;              // bytes per staged fp32 row
  static_assert(WN == 32 || WN % 64 == 0, "whole groups of 8 or 16 chunks");
  constexpr int SW = WN == 32 ? 7 : 15;     // chunks are XOR-permuted within groups of SW + 1
  constexpr int LPR = WN / 8;               // lanes per output row (8 columns each)
  constexpr int RPI = 64 / LPR;             // rows per store instruction
  constexpr int NSUB = 32 / RPI;            // store instructions per pass
  const int frow = lane & 31, fchunk = lane >> 5;
  const int rrow = lane / LPR, rcol = (lane % LPR) * 8;
  const int64_t col = col0 + J0 * 32 + rcol;
  auto inside = [&](int i, int sub) { return !EDGE || (row0 + i * 32 + sub * RPI + rrow < rows && col < cols); };   // (cols is a multiple of 8)
  bf16x8 bias = {}, aux[2][NSUB] = {};
  // (reads past the matrix are of its last row or columns: with a branch each they go out one by one, GeLU' 2000x6400x1600 57.7 / 53.3 us, 2944x9216x2304 142 / 134)
  const int64_t rcl = EDGE && col >= cols ? cols - 8 : col;
  if constexpr (epi_reads_bias(MODE)) bias = *reinterpret_cast<const bf16x8*>(epi.bias + rcl);
  auto fetch = [&](int i) {
#pragma unroll
    for (int sub = 0; sub < NSUB; ++sub) {
      const int64_t row = row0 + i * 32 + sub * RPI + rrow;
      aux[i & 1][sub] = *reinterpret_cast<const bf16x8*>(epi.aux_in + (EDGE && row >= rows ? rows - 1 : row) * epi.ldc + rcl);
    }
  };
  if constexpr (epi_reads_aux(MODE)) fetch(0);
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    if (epi_reads_aux(MODE) && i + 1 < TM) fetch(i + 1);
#pragma unroll
    for (int j = 0; j < WN / 32; ++j)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int c = j * 8 + g * 2 + fchunk;
        floatx4 v = {acc[i][J0 + j][g * 4 + 0], acc[i][J0 + j][g * 4 + 1], acc[i][J0 + j][g * 4 + 2], acc[i][J0 + j][g * 4 + 3]};
        *reinterpret_cast<floatx4*>(buf + frow * ROWB + (((c & ~SW) | ((c ^ frow) & SW)) << 4)) = v;
      }
    __builtin_amdgcn_s_waitcnt(DG_WAIT_LGKM0);  // own writes landed (the buffer is private to the wave)
#pragma unroll
    for (int sub = 0; sub < NSUB; ++sub) {
      const int r = sub * RPI + rrow, c0 = rcol / 4;
      const floatx4 lo = *reinterpret_cast<const floatx4*>(buf + r * ROWB + (((c0 & ~SW) | ((c0 ^ r) & SW)) << 4));
      const floatx4 hi = *reinterpret_cast<const floatx4*>(buf + r * ROWB + ((((c0 + 1) & ~SW) | (((c0 + 1) ^ r) & SW)) << 4));
      float v[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
      if (inside(i, sub)) gemm_epilogue8<MODE>(epi, row0 + i * 32 + r, col, v, bias, aux[i & 1][sub]);
    }
    __builtin_amdgcn_s_waitcnt(DG_WAIT_LGKM0);  // reads done before the next pass overwrites
  }
}

// Dynamic LDS of one workgroup: the operand stages, or the epilogue's per-wave staging where that is larger.
template <int BM, int BN, int WGM, int WGN, int MODE, int LS>
constexpr size_t dg_smem_bytes() {
  const size_t stages = (size_t)(LS == 5 ? 3 * (BM + BN) : (LS >= 2 ? 2 * BM + 3 * BN : DG_STAGES * (BM + BN))) * DG_BK * 2;
  const size_t pass = (size_t)WGM * WGN * 32 * (BN / WGN) * 4;   // 32 rows x WN floats per wave
  const size_t epi = (MODE == EPI_ACCUM_F32 || MODE == EPI_STORE_F32) ? 2 * pass : pass;
  return stages > epi ? stages : epi;
}

// LS (load schedule; 2, 4 and 5, with three stages of B or of both operands: in the body): 0 = the loads of a k-tile go out in one run right after the barrier that
// frees their stage (from the upper half of the waves, or from both halves one k-step apart,
// see below); 1 = every wave sends its share one load at a time between its products, spread
// over the three k-steps that follow that barrier, so that no wave sits at the texture
// addresser's full queue while its products wait.
// EDGE: M, N and K need not be multiples of the tile (rows, cols and K are the true extents; rows of both operands are
// whole 16-byte pieces).
template <int BM, int BN, int WGM, int WGN, bool A_KMAJOR, bool B_KMAJOR, int MODE, int LS, bool EDGE>
__device__ __forceinline__ void dg_tile(
    const bf16* __restrict__ a, int64_t lda, const bf16* __restrict__ b, int64_t ldb, int K,
    int tiles_m, int tiles_n, const EpiArgs<bf16>& epi, int group, int64_t rows, int64_t cols, int logical) {
  static_assert(!EDGE || LS == 4, "the other load schedules count loads that may lie outside an EDGE operand");
  constexpr int NW = WGM * WGN;
  constexpr int WM = BM / WGM, WN = BN / WGN;
  constexpr int TM = WM / 32, TN = WN / 32;
  // the epilogues swizzle 16-byte chunks of a staged fp32 row by the low four bits of the row
  // number, which needs rows of whole groups of 16 chunks (sub-tiles 96 wide are staged as 64 and 32)
  static_assert(WM % 32 == 0 && (WN % 64 == 0 || (WN == 96 && A_KMAJOR && B_KMAJOR)), "wave sub-tile: rows in 32s, columns in 64s or 96");
  constexpr int STAGE_ELEMS = (BM + BN) * DG_BK;
  extern __shared__ __attribute__((aligned(16))) unsigned char dg_smem[];
  bf16* smem = reinterpret_cast<bf16*>(dg_smem);  // [2][A tile | B tile]

  const int tid = threadIdx.x, lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int wm = wave / WGN, wn = wave % WGN;

  // Logical tile -> output tile, in groups of `group` tile rows.
  const int width = group * tiles_n;
  const int grp = logical / width;
  const int first_m = grp * group;
  const int gsize = (tiles_m - first_m < group) ? tiles_m - first_m : group;
  const int tile_m = first_m + (logical % width) % gsize;
  const int tile_n = (logical % width) / gsize;
  const int64_t m0 = (int64_t)tile_m * BM, n0 = (int64_t)tile_n * BN;

  // A direct load holds its wave at issue until the texture addresser takes it (about 20
  // cycles per 1 KB load, 64 loads per k-tile and CU), and a wave held there issues no
  // products.  With two waves per SIMD the loads are therefore arranged so that while one
  // wave of a SIMD is held at issue the other keeps the matrix pipe fed (measured per kernel):
  //   both operands k-major: only the upper half of the waves (one per SIMD) sends loads,
  //     the whole k-tile right after the barrier that frees the stage;
  //   an m/n-major operand: every wave sends its share, the lower half right after that
  //     barrier, the upper half one k-step later.
  // With one wave per SIMD every wave sends its share right after the barrier.
  constexpr bool HAND = !(A_KMAJOR && B_KMAJOR);
  constexpr bool SPLIT = (NW == 8) && HAND && LS == 0;          // two issue points
  constexpr int NI = (NW == 8 && !HAND && LS == 0) ? 4 : NW;    // number of issuing waves
  const bool issuer = wave >= NW - NI;
  const int iw = wave - (NW - NI);
  const bool early = !SPLIT || wave < NW / 2;
  DgLoader<BM, NI, A_KMAJOR, EDGE> la;
  DgLoader<BN, NI, B_KMAJOR, EDGE> lb;
  const int nkt = (K + DG_BK - 1) / DG_BK;   // k-tiles of the whole reduction
  const int k_tail = K - (nkt - 1) * DG_BK;
  la.init(a, lda, m0, issuer ? iw : 0, lane, (uint32_t)((A_KMAJOR ? (EDGE ? rows : (int64_t)tiles_m * BM) : (int64_t)K) * lda * 2), rows, k_tail, nkt - 1);
  lb.init(b, ldb, n0, issuer ? iw : 0, lane, (uint32_t)((B_KMAJOR ? (EDGE ? cols : (int64_t)tiles_n * BN) : (int64_t)K) * ldb * 2), cols, k_tail, nkt - 1);
  constexpr int LPT = DgLoader<BM, NI, A_KMAJOR, EDGE>::LPT + DgLoader<BN, NI, B_KMAJOR, EDGE>::LPT;

  floatx16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  // gridDim.y splits of the reduction (EPI_STORE_F32 only): this workgroup owns k-tiles kt0 .. kt0+nk-1
  int kt0 = 0, nk = nkt;
  if constexpr (MODE == EPI_STORE_F32) {
    kt0 = (int)(blockIdx.y * (unsigned)nkt / gridDim.y);
    nk = (int)((blockIdx.y + 1) * (unsigned)nkt / gridDim.y) - kt0;
  }
  // (opaque: bounds rewritten in terms of K cost the unrolled loop its compile-time knowledge of kt + 2 < nk)
  nk = __builtin_amdgcn_readfirstlane(nk);
  // Whether the loads of this workgroup's k-tile `kt` retire in order, so that a wait may count them: it exists, and
  // none of its loads lies outside the operand as a whole (a partly filled k-tile's may).
  auto counted = [&](int kt) { return kt < nk && (!EDGE || k_tail == DG_BK || kt0 + kt != nkt - 1); };
  // LDS map.  LS 0, 1: two stages of [A tile | B tile].  LS 2, 4: two stages of A, then three of B.  LS 5: three of A, three of B.
  constexpr int A_STRIDE = (LS >= 2) ? BM * DG_BK : STAGE_ELEMS;
  constexpr int B_STRIDE = (LS >= 2) ? BN * DG_BK : STAGE_ELEMS;
  constexpr int B_BASE = (LS >= 2) ? (LS == 5 ? 3 : 2) * BM * DG_BK : BM * DG_BK;
  // LS 2, 4: which of a wave's loads (A's LA first, then B's LB) go out in the k-step after the barrier
  // ([0, C3)), and in k-steps 0, 1, 2 of the next tile ([C3, C0), [C0, C1), [C1, LA+LB)).
  constexpr int LA_ = DgLoader<BM, NI, A_KMAJOR, EDGE>::LPT, LB_ = DgLoader<BN, NI, B_KMAJOR, EDGE>::LPT;
  // (Halves of A right after the barrier and in k-step 0, halves of B in k-steps 1 and 2; sending all of A
  // right after the barrier, or three quarters of it, measured the same to half a percent.)
  constexpr int C3 = LA_ / 2, C0 = LA_, C1 = LA_ + LB_ / 2;
  auto a_stage = [&](int i) { return smem + i * A_STRIDE; };
  auto b_stage = [&](int i) { return smem + B_BASE + i * B_STRIDE; };
  if constexpr (LS == 1) {
    // tile 0 whole; of tile 1 only the loads that in the steady state go out right after a
    // barrier -- the k-loop sends the rest during tile 0's first two k-steps, as for any tile
    constexpr int LA1 = DgLoader<BM, NI, A_KMAJOR, EDGE>::LPT, N31 = (LPT + 2) / 3;
    la.issue(smem, kt0, iw);
    lb.issue(smem + BM * DG_BK, kt0, iw);
    dg_static_for<N31>([&](auto j_tag) {
      constexpr int J = decltype(j_tag)::value;
      if constexpr (J < LA1) la.template issue_one<J>(smem + STAGE_ELEMS, kt0 + 1, iw, nk > 1);
      else lb.template issue_one<J - LA1>(smem + STAGE_ELEMS + BM * DG_BK, kt0 + 1, iw, nk > 1);
    });
    // (a load whose descriptor covers zero bytes makes no memory request and may retire ahead of
    // older loads still in flight: counting outstanding loads is only valid among live ones)
    if (nk > 1) __builtin_amdgcn_s_waitcnt(DG_WAIT_VM(N31)); else __builtin_amdgcn_s_waitcnt(DG_WAIT_VM(0));
  } else if constexpr (LS == 5) {
    la.issue(a_stage(0), kt0, iw);   // tile 0, then tile 1 (past the end: zeros, as below)
    lb.issue(b_stage(0), kt0, iw);
    dg_static_for<LA_>([&](auto j_tag) { la.template issue_one<decltype(j_tag)::value>(a_stage(1), kt0 + 1, iw, nk > 1); });
    dg_static_for<LB_>([&](auto j_tag) { lb.template issue_one<decltype(j_tag)::value>(b_stage(1), kt0 + 1, iw, nk > 1); });
    if (counted(1)) __builtin_amdgcn_s_waitcnt(DG_WAIT_VM(LA_ + LB_)); else __builtin_amdgcn_s_waitcnt(DG_WAIT_VM(0));
  } else if constexpr (LS >= 2) {
    // A(0), B(0) whole, then B(1) whole and the loads of tile 1 that go out right after a barrier (all of
    // them A's): what the steady state has sent for tile 0's period by the time its k-step 0 starts.
    static_assert(C3 <= LA_ && C0 >= LA_, "only A's loads follow the barrier; A is complete after k-step 0");
    la.issue(a_stage(0), kt0, iw);
    lb.issue(b_stage(0), kt0, iw);
    dg_static_for<LB_>([&](auto j_tag) { lb.template issue_one<decltype(j_tag)::value>(b_stage(1), kt0 + 1, iw, nk > 1); });
    dg_static_for<C3>([&](auto j_tag) { la.template issue_one<decltype(j_tag)::value>(a_stage(1), kt0 + 1, iw, nk > 1); });
    if (counted(1)) __builtin_amdgcn_s_waitcnt(DG_WAIT_VM(LB_ + C3)); else __builtin_amdgcn_s_waitcnt(DG_WAIT_VM(0));
  } else if (issuer) {
    la.issue(smem, kt0, iw);
    lb.issue(smem + BM * DG_BK, kt0, iw);
    if (nk > 1) {
      la.issue(smem + STAGE_ELEMS, kt0 + 1, iw);
      lb.issue(smem + STAGE_ELEMS + BM * DG_BK, kt0 + 1, iw);
      __builtin_amdgcn_s_waitcnt(DG_WAIT_VM(LPT));  // tile 0 landed, tile 1 may be in flight
    } else {
      __builtin_amdgcn_s_waitcnt(DG_WAIT_VM(0));
    }
  }
  __builtin_amdgcn_s_barrier();

  DgFragReg<A_KMAJOR, HAND> fa[2][TM];
  DgFragReg<B_KMAJOR, HAND> fb[2][TN];
  static_assert(WM % 32 == 0 && WN % 32 == 0, "the fragment readers take a wave's first row as a multiple of 32");
  using KS0 = std::integral_constant<int, 0>;
  using KS1 = std::integral_constant<int, 1>;
  using KS2 = std::integral_constant<int, 2>;
  using KS3 = std::integral_constant<int, 3>;
  dg_static_for<TN>([&](auto j) { DgFrag<BN, B_KMAJOR, HAND>::fetch(fb[0][decltype(j)::value], b_stage(0), wn * WN, j, KS0{}, lane); });
  dg_static_for<TM>([&](auto i) { DgFrag<BM, A_KMAJOR, HAND>::fetch(fa[0][decltype(i)::value], a_stage(0), wm * WM, i, KS0{}, lane); });

  constexpr int NMFMA = TM * TN;
  constexpr int NREAD = (A_KMAJOR ? TM : 2 * TM) + (B_KMAJOR ? TN : 2 * TN);
  constexpr int RPM = (NREAD + NMFMA - 1) / NMFMA;
  using S0 = std::integral_constant<int, 0>;
  using S1 = std::integral_constant<int, 1>;

  if constexpr (LS == 0) {
  // One k-step of 16: multiply fragment set `cur` while set `cur^1` is fetched from
  // (tile, ks_next).  The hints pin the order MFMA, LDS read, MFMA, LDS read, ... so the
  // LDS latency hides behind the matrix pipe.
  auto kstep = [&](auto cur_tag, const bf16* ta, auto ks_next) {
    constexpr int cur = decltype(cur_tag)::value;
    const bf16* tb = ta + BM * DG_BK;
    // hand-waited fragments of set `cur` (fetched during the previous k-step) first, so the
    // wait does not cover the reads issued next
    dg_settle_all(fb[cur]);
    dg_settle_all(fa[cur]);
    dg_static_for<TN>([&](auto j) { DgFrag<BN, B_KMAJOR, HAND>::fetch(fb[cur ^ 1][decltype(j)::value], tb, wn * WN, j, ks_next, lane); });
    dg_static_for<TM>([&](auto i) { DgFrag<BM, A_KMAJOR, HAND>::fetch(fa[cur ^ 1][decltype(i)::value], ta, wm * WM, i, ks_next, lane); });
    // hand-issued reads go out before this k-step's products, so they have the whole k-step to land
    if constexpr (HAND) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(dg_value(fb[cur][j]), dg_value(fa[cur][i]), acc[i][j], 0, 0, 0);
    if constexpr (!HAND) DgInterleave<0, NMFMA, NREAD, RPM, 0>::hint();
    else __builtin_amdgcn_sched_barrier(0);  // the products stay above the next k-step's wait
  };

  // Per k-tile kt (stage kt&1):
  //   k-steps 0..2 multiply while fetching the next k-step's fragments from the same tile;
  //   then every wave waits for its own reads and for its share of tile kt+1 to land, and
  //   the workgroup barrier makes both facts global: tile kt's stage may now be refilled
  //   (tile kt+2 is issued into it) and tile kt+1 may be read;
  //   k-step 3 multiplies while fetching k-step 0 of tile kt+1 (on the last tile that is a
  //   stale but in-bounds read whose result is never used).
  for (int kt = 0; kt < nk; ++kt) {
    bf16* cur = smem + (kt & 1) * STAGE_ELEMS;
    bf16* nxt = smem + ((kt & 1) ^ 1) * STAGE_ELEMS;
    kstep(S0{}, cur, KS1{});
    if (SPLIT && !early && kt >= 1 && kt + 1 < nk) {  // the late half's share of tile kt+1 (tiles 0, 1: sent above)
      la.issue(nxt, kt0 + kt + 1, iw);
      lb.issue(nxt + BM * DG_BK, kt0 + kt + 1, iw);
    }
    kstep(S1{}, cur, KS2{});
    kstep(S0{}, cur, KS3{});
    __builtin_amdgcn_s_waitcnt(DG_WAIT_VM0_LGKM0);
    __builtin_amdgcn_s_barrier();
    if (issuer && early && kt + 2 < nk) {
      la.issue(cur, kt0 + kt + 2, iw);
      lb.issue(cur + BM * DG_BK, kt0 + kt + 2, iw);
    }
    kstep(S1{}, nxt, KS0{});
  }
  } else {
  // Loads sent one at a time between products.  A wave's LT loads of a k-tile are numbered A's
  // first (LA of them), then B's.
  //   LS 1: those numbered [0, N3) go out in the k-step after the barrier that frees their stage,
  //     [N3, N3+N0) and the rest in the two k-steps after it; the k-step before the next barrier
  //     carries none, so the last ones have that long to land.
  //   LS 2: B has a third stage, so B's loads for tile kt+2 can go out while tile kt is still being
  //     read: every k-step carries the same number of loads (A's halves in the k-step after the
  //     barrier and the one after it, B's halves in the other two) and the path from L2 into LDS,
  //     which is what bounds a 256x256 tile, never runs dry between barriers.
  constexpr int LA = DgLoader<BM, NI, A_KMAJOR, EDGE>::LPT, LB = DgLoader<BN, NI, B_KMAJOR, EDGE>::LPT, LT = LPT;
  constexpr int N3 = (LT + 2) / 3, N0 = (LT - N3 + 1) / 2;
  auto kstep = [&](auto cur_tag, const bf16* ta, const bf16* tb, auto ks_next, auto loads, bf16* lda_stage, int lda_kt,
                   bool lda_live, bf16* ldb_stage, int ldb_kt, bool ldb_live) {
    constexpr int cur = decltype(cur_tag)::value;
    constexpr int LO = decltype(loads)::lo, HI = decltype(loads)::hi;
    dg_settle_all(fb[cur]);
    dg_settle_all(fa[cur]);
    auto fetch_one = [&](auto r_tag) {   // read number r of the next k-step's fragments: B's first, then A's
      constexpr int R = decltype(r_tag)::value;
      if constexpr (R < TN) DgFrag<BN, B_KMAJOR, HAND>::fetch(fb[cur ^ 1][R], tb, wn * WN, std::integral_constant<int, R>{}, ks_next, lane);
      else DgFrag<BM, A_KMAJOR, HAND>::fetch(fa[cur ^ 1][R - TN], ta, wm * WM, std::integral_constant<int, R - TN>{}, ks_next, lane);
    };
    if constexpr (HAND) {
      dg_static_for<TM + TN>(fetch_one);
      __builtin_amdgcn_sched_barrier(0);
    }
    dg_static_for<NMFMA>([&](auto q_tag) {
      constexpr int Q = decltype(q_tag)::value, I = Q / TN, J = Q % TN;
      acc[I][J] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(dg_value(fb[cur][J]), dg_value(fa[cur][I]), acc[I][J], 0, 0, 0);
      if constexpr (!HAND) {   // source order = the order the hints ask for: product, fragment read(s), load
        constexpr int FR = (TM + TN + NMFMA - 1) / NMFMA;   // fragments per product
        dg_static_for<FR>([&](auto f_tag) {
          constexpr int R = Q * FR + decltype(f_tag)::value;
          if constexpr (R < TM + TN) fetch_one(std::integral_constant<int, R>{});
        });
      }
      if constexpr (HI > LO) {
        dg_static_for<HI - LO>([&](auto l_tag) {
          constexpr int L = LO + decltype(l_tag)::value;
          if constexpr (dg_load_slot(L, LO, HI, NMFMA) == Q) {
            if constexpr (HAND) __builtin_amdgcn_sched_barrier(0);
            if constexpr (L < LA) la.template issue_one<L>(lda_stage, lda_kt, iw, lda_live);
            else lb.template issue_one<L - LA>(ldb_stage, ldb_kt, iw, ldb_live);
            if constexpr (HAND) __builtin_amdgcn_sched_barrier(0);
          }
        });
      }
    });
    if constexpr (!HAND) DgInterleaveMask<0, NMFMA, NREAD, RPM, (HI > LO ? dg_load_mask(LO, HI, NMFMA) : 0u)>::hint();
    else __builtin_amdgcn_sched_barrier(0);
  };
  if constexpr (LS == 1) {
    for (int kt = 0; kt < nk; ++kt) {
      bf16* cur = smem + (kt & 1) * STAGE_ELEMS;
      bf16* nxt = smem + ((kt & 1) ^ 1) * STAGE_ELEMS;
      bf16* curb = cur + BM * DG_BK;
      bf16* nxtb = nxt + BM * DG_BK;
      // A load for a k-tile past the end deposits zeros into a stage nobody reads any more.
      const bool live_next = kt + 1 < nk;   // tile kt+1's remaining loads
      kstep(S0{}, cur, curb, KS1{}, DgLoads<N3, N3 + N0>{}, nxt, kt0 + kt + 1, live_next, nxtb, kt0 + kt + 1, live_next);
      kstep(S1{}, cur, curb, KS2{}, DgLoads<N3 + N0, LT>{}, nxt, kt0 + kt + 1, live_next, nxtb, kt0 + kt + 1, live_next);
      kstep(S0{}, cur, curb, KS3{}, DgLoads<0, 0>{}, nxt, 0, false, nxtb, 0, false);
      __builtin_amdgcn_s_waitcnt(DG_WAIT_VM0_LGKM0);
      __builtin_amdgcn_s_barrier();
      kstep(S1{}, nxt, nxtb, KS0{}, DgLoads<0, N3>{}, cur, kt0 + kt + 2, kt + 2 < nk, curb, kt0 + kt + 2, kt + 2 < nk);
    }
  } else if constexpr (LS == 5) {
    // Three stages of both operands: all loads of tile kt+2 go into the stage of tile kt-1, a quarter in every k-step.
    constexpr int L1 = LT / 4, L2 = LT / 2, L3 = 3 * LT / 4;
    auto ktile = [&](auto s_tag, int kt) {
      constexpr int P = decltype(s_tag)::value, P1 = (P + 1) % 3, P2 = (P + 2) % 3;
      bf16* ca = a_stage(P);
      bf16* cb = b_stage(P);
      bf16* fa2 = a_stage(P2);
      bf16* fb2 = b_stage(P2);
      const bool live = kt + 2 < nk;
      kstep(S0{}, ca, cb, KS1{}, DgLoads<0, L1>{}, fa2, kt0 + kt + 2, live, fb2, kt0 + kt + 2, live);
      kstep(S1{}, ca, cb, KS2{}, DgLoads<L1, L2>{}, fa2, kt0 + kt + 2, live, fb2, kt0 + kt + 2, live);
      kstep(S0{}, ca, cb, KS3{}, DgLoads<L2, L3>{}, fa2, kt0 + kt + 2, live, fb2, kt0 + kt + 2, live);
      // tile kt+1 must have landed; the L3 loads of tile kt+2 sent so far may be in flight (see the LS 2 loop)
      if (counted(kt + 2)) __builtin_amdgcn_s_waitcnt(DG_WAIT_VM(L3) & DG_WAIT_LGKM0);
      else __builtin_amdgcn_s_waitcnt(DG_WAIT_VM0_LGKM0);
      __builtin_amdgcn_s_barrier();
      kstep(S1{}, a_stage(P1), b_stage(P1), KS0{}, DgLoads<L3, LT>{}, fa2, kt0 + kt + 2, live, fb2, kt0 + kt + 2, live);
    };
    using S2 = std::integral_constant<int, 2>;
    int kt = 0;
    for (; kt + 3 <= nk; kt += 3) {
      ktile(S0{}, kt);
      ktile(S1{}, kt + 1);
      ktile(S2{}, kt + 2);
    }
    if (kt < nk) { ktile(S0{}, kt); ++kt; }
    if (kt < nk) { ktile(S1{}, kt); ++kt; }
  } else {
    // One k-tile whose A stage AP (kt mod 2) and B stage BS (kt mod 3) are compile-time values.
    auto ktile = [&](auto ap_tag, auto bs_tag, int kt) {
      constexpr int AP = decltype(ap_tag)::value, BS = decltype(bs_tag)::value;
      constexpr int BS1 = (BS + 1) % 3, BS2 = (BS + 2) % 3;
      bf16* ca = a_stage(AP);
      bf16* na = a_stage(AP ^ 1);
      bf16* cb = b_stage(BS);
      bf16* nb = b_stage(BS1);
      bf16* nnb = b_stage(BS2);   // held tile kt-1: free since the last barrier
      const bool live1 = kt + 1 < nk, live2 = kt + 2 < nk;
      kstep(S0{}, ca, cb, KS1{}, DgLoads<C3, C0>{}, na, kt0 + kt + 1, live1, nnb, kt0 + kt + 2, live2);
      kstep(S1{}, ca, cb, KS2{}, DgLoads<C0, C1>{}, na, 0, false, nnb, kt0 + kt + 2, live2);
      kstep(S0{}, ca, cb, KS3{}, DgLoads<C1, LT>{}, na, 0, false, nnb, kt0 + kt + 2, live2);
      if (counted(kt + 2)) __builtin_amdgcn_s_waitcnt(DG_WAIT_VM(LB) & DG_WAIT_LGKM0);   // (see the loop below)
      else __builtin_amdgcn_s_waitcnt(DG_WAIT_VM0_LGKM0);
      __builtin_amdgcn_s_barrier();
      kstep(S1{}, na, nb, KS0{}, DgLoads<0, C3>{}, ca, kt0 + kt + 2, live2, nnb, 0, false);
    };
    using S2 = std::integral_constant<int, 2>;
    if constexpr (LS == 4) {
      // The loop unrolled over the period of the stage pair (2 x 3 k-tiles): every LDS address of a
      // fragment read or a load's destination is then a lane-dependent register plus a constant, and
      // the address arithmetic that otherwise follows the stage pointers around the loop (about one
      // vector and one scalar instruction per product) is gone.
      int kt = 0;
      for (; kt + 6 <= nk; kt += 6) {
        ktile(S0{}, S0{}, kt);
        ktile(S1{}, S1{}, kt + 1);
        ktile(S0{}, S2{}, kt + 2);
        ktile(S1{}, S0{}, kt + 3);
        ktile(S0{}, S1{}, kt + 4);
        ktile(S1{}, S2{}, kt + 5);
      }
      if (kt < nk) { ktile(S0{}, S0{}, kt); ++kt; }
      if (kt < nk) { ktile(S1{}, S1{}, kt); ++kt; }
      if (kt < nk) { ktile(S0{}, S2{}, kt); ++kt; }
      if (kt < nk) { ktile(S1{}, S0{}, kt); ++kt; }
      if (kt < nk) { ktile(S0{}, S1{}, kt); ++kt; }
    } else {
      int bs = 0;   // B stage of tile kt (kt mod 3)
      for (int kt = 0; kt < nk; ++kt) {
        bf16* ca = a_stage(kt & 1);
        bf16* na = a_stage((kt & 1) ^ 1);
        const int bs1 = bs == 2 ? 0 : bs + 1, bs2 = bs1 == 2 ? 0 : bs1 + 1;
        bf16* cb = b_stage(bs);
        bf16* nb = b_stage(bs1);
        bf16* nnb = b_stage(bs2);   // held tile kt-1: free since the last barrier
        const bool live1 = kt + 1 < nk, live2 = kt + 2 < nk;
        kstep(S0{}, ca, cb, KS1{}, DgLoads<C3, C0>{}, na, kt0 + kt + 1, live1, nnb, kt0 + kt + 2, live2);
        kstep(S1{}, ca, cb, KS2{}, DgLoads<C0, C1>{}, na, 0, false, nnb, kt0 + kt + 2, live2);
        kstep(S0{}, ca, cb, KS3{}, DgLoads<C1, LT>{}, na, 0, false, nnb, kt0 + kt + 2, live2);
        // tile kt+1 must have landed (A's second half went out three k-steps ago, B's a period ago); the
        // LB loads of B(kt+2) sent since then may still be in flight.  That count holds only while
        // those loads are live: past the end of the reduction they make no memory request and may
        // retire ahead of older loads, so the last two k-tiles wait for everything.
        if (live2) __builtin_amdgcn_s_waitcnt(DG_WAIT_VM(LB) & DG_WAIT_LGKM0);
        else __builtin_amdgcn_s_waitcnt(DG_WAIT_VM0_LGKM0);
        __builtin_amdgcn_s_barrier();
        kstep(S1{}, na, nb, KS0{}, DgLoads<0, C3>{}, ca, kt0 + kt + 2, live2, nnb, 0, false);
        bs = bs1;
      }
    }
  }
  }

  const int frow = lane & 31, fchunk = lane >> 5;
  if constexpr (MODE == EPI_ACCUM_F32 || MODE == EPI_STORE_F32) {
    // out_f32 += acc.  Reading the old values through registers would leave only a few KB
    // in flight per CU (the accumulators own the register file), so the old tile is
    // streamed into the now idle LDS with the same direct loads as the operands: each wave
    // pulls its own sub-tile in passes of 32 rows x WN floats, double-buffered, adds its
    // accumulators in place and stores the sums out of LDS, consecutive lanes along a row.  Chunks of 16 B are
    // XOR-swizzled by the row so that 16 lanes reading one column of 16 rows hit distinct banks.
    // Bound by memory (old values in, sums out).  Stored straight from the accumulators' layout an instruction wrote 32 bytes of
    // each of 32 rows; as whole rows, before / after (us, += over 2048 tokens, operands out of cache): 12288x3072 210 / 196 on 256x256
    // tiles, 194 / 188 on 128x128; 4096^2 84 / 79, 91 / 88; 8192^2 340 / 322, 333 / 323.  Without any epilogue 12288x3072 takes
    // 143 and 140, and 302 MB in and out take 66 by themselves.  Slower still: stores past the caches, fp32 atomics, more passes in registers.
    constexpr int CPR = WN / 4;                 // 16-byte chunks per row of the pass block
    constexpr int PASS_BYTES = 32 * WN * 4;
    constexpr int NINS = PASS_BYTES / 1024;     // direct loads per pass
    static_assert(NW * 2 * PASS_BYTES <= dg_smem_bytes<BM, BN, WGM, WGN, MODE, LS>(), "epilogue staging must fit the workgroup's LDS");
    __builtin_amdgcn_s_waitcnt(DG_WAIT_VM0_LGKM0);
    __builtin_amdgcn_s_barrier();               // every wave is done with the operand stages
    unsigned char* mybuf = dg_smem + wave * (2 * PASS_BYTES);
    float* cbase = epi.out_f32 + (MODE == EPI_STORE_F32 ? (int64_t)blockIdx.y * epi.split_stride : 0) +
                   (m0 + wm * WM) * epi.ldc + n0 + wn * WN;
    // from the sub-tile's first row and column to the end of the matrix; both may be negative when it lies outside
    const int64_t rows_left = rows - (m0 + wm * WM), cols_left = cols - (n0 + wn * WN);
    auto issue_pass = [&](int pass) {
      unsigned char* buf = mybuf + (pass & 1) * PASS_BYTES;
#pragma unroll
      for (int q = 0; q < NINS; ++q) {
        const int slot = q * 64 + lane, row = slot / CPR, pc = slot % CPR;
        const int c = pc ^ (row & 15);
        int64_t gr = pass * 32 + row, gc = c * 4;
        if constexpr (EDGE) {   // outside the matrix: some element inside it (what is loaded there is not stored)
          gr = gr < rows_left ? gr : rows_left - 1;
          gc = gc < cols_left ? gc : cols_left - 4;
        }
        __builtin_amdgcn_global_load_lds((glb_ptr_t)(cbase + gr * epi.ldc + gc), (lds_ptr_t)(buf + q * 1024), 16, 0, 0);
      }
    };
    if constexpr (MODE == EPI_ACCUM_F32) {
      issue_pass(0);
      if (TM > 1) issue_pass(1);
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      if constexpr (MODE == EPI_ACCUM_F32) {
        if (i + 1 < TM) __builtin_amdgcn_s_waitcnt(DG_WAIT_VM(NINS)); else __builtin_amdgcn_s_waitcnt(DG_WAIT_VM(0));
      }
      unsigned char* buf = mybuf + (i & 1) * PASS_BYTES;
      float* crow = cbase + (int64_t)(i * 32 + frow) * epi.ldc;
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int c = j * 8 + g * 2 + fchunk;
          floatx4* slot = reinterpret_cast<floatx4*>(buf + frow * (WN * 4) + ((c ^ (frow & 15)) << 4));
          floatx4 v = {0.f, 0.f, 0.f, 0.f};   // EPI_STORE_F32: a partial sum of its own, nothing to add to
          if constexpr (MODE == EPI_ACCUM_F32) v = *slot;
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] += acc[i][j][g * 4 + e];
          if constexpr (MODE == EPI_ACCUM_F32) *slot = v;
          else if (!EDGE || (i * 32 + frow < rows_left && c * 4 < cols_left)) *reinterpret_cast<floatx4*>(crow + c * 4) = v;
        }
      if constexpr (MODE == EPI_ACCUM_F32) {
        __builtin_amdgcn_s_waitcnt(DG_WAIT_LGKM0);
#pragma unroll
        for (int q = 0; q < NINS; ++q) {
          const int slot = q * 64 + lane, row = slot / CPR, c = slot % CPR;
          const floatx4 v = *reinterpret_cast<const floatx4*>(buf + row * (WN * 4) + ((c ^ (row & 15)) << 4));
          if (!EDGE || (i * 32 + row < rows_left && c * 4 < cols_left))
            *reinterpret_cast<floatx4*>(cbase + (int64_t)(i * 32 + row) * epi.ldc + c * 4) = v;
        }
      }
      if (MODE == EPI_ACCUM_F32 && i + 2 < TM) {
        __builtin_amdgcn_s_waitcnt(DG_WAIT_LGKM0);  // this buffer's LDS reads are done before it is refilled
        issue_pass(i + 2);
      }
    }
  } else {
    // bf16 outputs.  acc[i][j][r] is row m = lane%32 of the 32x32 tile, column
    // n = 8*(r/4) + 4*(lane/32) + r%4: storing straight from that layout writes 8-byte
    // pieces of many rows per instruction and was measured to amplify HBM write traffic
    // 2-3x.  Instead each wave transposes its sub-tile through the idle LDS, 32 rows at a
    // time (fp32, chunk-XOR-swizzled), and re-reads it with consecutive lanes along a row,
    // so bias / residual / pre-GeLU reads and all stores are 16 bytes per lane and whole
    // 128-byte lines per row.
    static_assert(NW * 32 * WN * 4 <= dg_smem_bytes<BM, BN, WGM, WGN, MODE, LS>(), "epilogue staging must fit the workgroup's LDS");
    __builtin_amdgcn_s_waitcnt(DG_WAIT_VM0_LGKM0);
    __builtin_amdgcn_s_barrier();             // every wave is done with the operand stages
    if constexpr (WN % 64 == 0) {
      dg_epilogue_bf16<MODE, TM, TN, WN, EDGE>(acc, dg_smem + wave * (32 * WN * 4), epi, m0 + wm * WM, n0 + wn * WN, lane, rows, cols);
    } else {
      dg_epilogue_bf16<MODE, TM, TN, 64, EDGE>(acc, dg_smem + wave * (32 * WN * 4), epi, m0 + wm * WM, n0 + wn * WN, lane, rows, cols);
      dg_epilogue_bf16<MODE, TM, TN, 32, EDGE, 2>(acc, dg_smem + wave * (32 * WN * 4), epi, m0 + wm * WM, n0 + wn * WN, lane, rows, cols);
    }
  }
}

// Workgroup -> tile.  Consecutive workgroup ids go round-robin over the 8 XCDs; give every XCD a contiguous range of
// logical tiles, walked in groups of tile rows so the A and B panels an XCD touches stay in its L2.
template <int BM, int BN, int WGM, int WGN, bool A_KMAJOR, bool B_KMAJOR, int MODE, int LS = 0, bool EDGE = false>
__global__ __launch_bounds__(WGM* WGN* kWave) void gemm_dma_kernel(
    const bf16* __restrict__ a, int64_t lda, const bf16* __restrict__ b, int64_t ldb, int K,
    int tiles_m, int tiles_n, EpiArgs<bf16> epi, int xcd_remap, int group, int64_t rows, int64_t cols) {
  int logical = blockIdx.x;
  const int nblk = gridDim.x;
  if (xcd_remap && (nblk & 7) == 0) logical = (blockIdx.x & 7) * (nblk >> 3) + (blockIdx.x >> 3);
  dg_tile<BM, BN, WGM, WGN, A_KMAJOR, B_KMAJOR, MODE, LS, EDGE>(a, lda, b, ldb, K, tiles_m, tiles_n, epi, group, rows, cols, logical);
}

// Several weight gradients out[M,N] += a[K,M]^T b[K,N] over the same K in one launch.  Alone each of them ends with a
// partly filled round of workgroups (or leaves slots empty throughout); together only the last one does.
// Job j owns workgroups first[j] .. first[j+1]-1, a multiple of 8 of them, remapped among themselves as above; those
// past its last tile end at once.
typedef WgradJob<bf16> DgJob;
struct DgGroup {
  int n, K;
  int first[kMaxGroupJobs + 1];
  DgJob job[kMaxGroupJobs];
};
template <int BM, int BN, int WGM, int WGN, bool EDGE>
__global__ __launch_bounds__(WGM* WGN* kWave) void gemm_group_kernel(DgGroup g, int group) {
  int j = 0;
  while (j + 1 < g.n && (int)blockIdx.x >= g.first[j + 1]) ++j;
  const DgJob& w = g.job[j];
  const int local = (int)blockIdx.x - g.first[j], nblk = g.first[j + 1] - g.first[j];
  const int logical = (local & 7) * (nblk >> 3) + (local >> 3);
  const int tiles_m = (w.M + BM - 1) / BM, tiles_n = (w.N + BN - 1) / BN;
  if (logical >= tiles_m * tiles_n) return;
  const EpiArgs<bf16> epi{nullptr, nullptr, nullptr, nullptr, w.out, w.N, DropArgs{}, 0};
  dg_tile<BM, BN, WGM, WGN, false, false, EPI_ACCUM_F32, 4, EDGE>(w.a, w.M, w.b, w.N, g.K, tiles_m, tiles_n, epi, group, w.M, w.N, logical);
}

// ---------------------------------------------------------------------------
// host side.  Variant ids (0 is "the library's choice", -1 the kernels of gemm_cut.h):
//   5: 256x256 tile, 8 waves   6: 256x256, 4 waves   7: 128x128, 4 waves   8: 256x128, 4 waves
//   9: as 5 with the spread load schedule   10: as 7 with the spread load schedule   11: as 6 with it
//   12: as 5 with three stages of B and loads in every k-step   13: as 6 with that   14: as 7 with that
//   15: 128x256, 8 waves, that schedule   16: 256x128, 8 waves, that schedule
//   17: as 13 with the k-tile loop unrolled over the stage period   18: as 12 with that
//   19: as 14 with that
//   20: 128x256, 21: 256x128, 4 waves, three stages of both operands (LS 5)
//   24: 128x192 in that form, forward only; the library takes it in place of 20 where dg_narrow says so
//   22, 23: as 19, 18 for sizes that are no multiples of the tile (EDGE)
// dg_pick and dg_group_choice go by the tiles' rounds (the debug queries _choice); dg_at_launch and dg_group_wide may take another configuration when the
// product is launched (the queries _launch).
// ---------------------------------------------------------------------------
inline bool dg_variant_tile(int variant, GemmTile* t) {
  switch (variant) {
    case 5: case 6: case 9: case 11: case 12: case 13: case 17: case 18: case 23: *t = {256, 256}; return true;
    case 7: case 10: case 14: case 19: case 22: *t = {128, 128}; return true;
    case 8: case 16: case 21: *t = {256, 128}; return true;
    case 15: case 20: *t = {128, 256}; return true;
    case 24: *t = {128, 192}; return true;
    default: return false;
  }
}

inline bool dg_shape_ok(int variant, int64_t M, int64_t N, int64_t K, int64_t lda, int64_t ldb) {
  GemmTile t;
  if (!dg_variant_tile(variant, &t)) return false;
  // operands are addressed with 32-bit byte offsets from their base (buffer loads)
  const int64_t a_bytes = (M > K ? M : K) * lda * 2, b_bytes = (N > K ? N : K) * ldb * 2;
  if (variant == 22 || variant == 23) {   // EDGE: rows of both operands and of the output are whole 16-byte pieces; offsets below DG_OUTSIDE
    const int64_t pad = 2 * 256 * (lda > ldb ? lda : ldb);
    return lda % 8 == 0 && ldb % 8 == 0 && N % 8 == 0 && K >= 1 && ((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn) < (1ll << 31) &&
           a_bytes + pad < DG_OUTSIDE && b_bytes + pad < DG_OUTSIDE;
  }
  return M % t.bm == 0 && N % t.bn == 0 && K % DG_BK == 0 && K >= DG_BK && lda % 8 == 0 && ldb % 8 == 0 &&
         (M / t.bm) * (N / t.bn) < (1ll << 31) && a_bytes < (1ll << 32) && b_bytes < (1ll << 32);
}

// The merged 128x256 and 256x128 tiles run on four waves (64x128 / 128x64 each: 6 fragment reads per 8 products), not on eight
// of 64x64 (4 per 4): with eight the LDS moves 128 KB of fragments and 48 KB of new data per k-tile, 1400 clocks against
// 1024 of products.  Eight against four waves on operands out of cache (us): forward 2048x3072x12288 186 / 169, 2048x12288x3072
// 158 / 150; dgrad 2048x3072x9216 138 / 126; on 256x128 219 / 183, 167 / 153, 168 / 141.  The LDS (160 KB) holds a third stage
// of A as well (LS 5: 144 KB), which gives every load two k-tiles to arrive and the loop a period of three: again (us, forward / dgrad)
// 169 / 174 -> 164 / 161 at 2048x3072x12288, 126 / 126 -> 123 / 119 at 2048x3072x9216, on 256x128 183 / 187 -> 170 / 161.  (128x128 tiles on two waves of
// 128x64: 3-15 % faster than on four with cached operands, 3-10 % slower otherwise.)
// Picks between the 256x256 (one workgroup per CU) and 128x128 (two per CU) tiles by the
// number of full-chip rounds each needs; 0 if neither fits the shape.  Sizes that are no multiples of 128 (64 for K)
// take the EDGE form of the same two tiles, if their rows are whole 16-byte pieces and the product is larger than one
// tile (which gemm_cut.h cuts into 16 or more workgroups; so it does with products of few tiles, dg_cut_sooner).  Against
// fp32 products (us, forward / dgrad / wgrad): 2000x1600x1600 184 / 161 / 147 -> 18 / 18 / 22 on 128x128 (34 on 256x256),
// 2000x6400x1600 495 / 481 / 509 -> 42 / 43 / 54 on 256x256 (50 on 128x128).  At sizes both forms take the plain one is
// 1-5 % faster.
inline int dg_choose_variant(int64_t M, int64_t N, int64_t K, int64_t lda, int64_t ldb) {
  const bool ok5 = dg_shape_ok(5, M, N, K, lda, ldb), ok7 = dg_shape_ok(7, M, N, K, lda, ldb);
  const bool edge = !ok7;   // anything divisible by 256 is divisible by 128
  if (edge && !(dg_shape_ok(22, M, N, K, lda, ldb) && (M > 128 || N > 128))) return 0;
  if (ok7 && !ok5) return 7;
  const int64_t t5 = ((M + 255) / 256) * ((N + 255) / 256), t7 = ((M + 127) / 128) * ((N + 127) / 128);
  const double cost5 = (double)((t5 + 255) / 256) * 4.0 / 1.15;
  const double cost7 = (double)((t7 + 511) / 512) * 2.0;
  if (edge) return cost5 <= cost7 ? 23 : 22;
  return cost5 <= cost7 ? 5 : 7;
}

// Kernel configuration for a product once the tile size is chosen (tile_variant 5: 256x256, 7:
// 128x128), picked by timing whole stage steps with each combination in one process (the chip
// runs the step at its board power limit, so what counts is energy per product, not the rate of
// a kernel alone): the 256x256 forward product runs on 4 waves (128x128 per wave: a third fewer
// LDS reads per product) with a third B stage and loads in every k-step; dgrad keeps 8 waves
// (two per SIMD hide each other's waits on the two-instruction transposed reads) with the same
// load schedule, and so does wgrad (both operands read transposed); all of them with the k-tile
// loop unrolled over the stage period, which removes the address arithmetic from the loop and was
// worth 4.4 % of the C5 step and 1.4-2.6 % of the smaller stages' in same-process A/B.
struct DgFlavours { int fwd256 = 17, bwd256 = 18, fwd128 = 19, dgrad128 = 19, wgrad128 = 19, wgrad256 = 18; bool pair128 = true, group = true, named = false, small[3] = {true, true, true}; };
inline DgFlavours& dg_flavours() { static DgFlavours f; return f; }   // tuning hook: varuna_debug_set_gemm_kernels
inline int dg_flavour(int tile_variant, int op) {
  const DgFlavours& f = dg_flavours();
  if (tile_variant == 5) return op == GEMM_FWD ? f.fwd256 : (op == GEMM_DGRAD ? f.bwd256 : f.wgrad256);
  if (tile_variant == 7) return op == GEMM_FWD ? f.fwd128 : (op == GEMM_DGRAD ? f.dgrad128 : f.wgrad128);
  return tile_variant;
}

// Whether a product of so few 128x128 tiles that most CUs would stay idle ends sooner on the small tiles of gemm_cut.h, whose waves share
// the reduction.  Measured back to back, this kernel / those (us, forward, dgrad, wgrad): 512x512 over 512 6.8 / 4.3, 6.3 / 5.2, 7.9 / 6.6,
// over 1024 8.9 / 5.0, 8.8 / 6.3, 10.6 / 8.2, over 4096 36 / 17 (wgrad); 512x1024 over 512 7.0 / 5.5, 6.4 / 6.5, 8.1 / 8.3, over 1024 9.4 / 7.4, 9.6 / 8.7, 13.6 / 12.1;
// 1024^2 over 1024 12.3 / 11.3, 12.2 / 11.1, 14.0 / 18.3 and over 4096 1.4, 1.6 and 1.2 times as fast; at 96 tiles always slower.
// The lines are those of operands in cache and keep off where the two are close there (1024^2 over 1024 on a later measurement 8.9 / 10.1,
// 8.8 / 9.4, 11.0 / 14.9).  With operands out of cache the small tiles are ahead further up in forward and dgrad: 1024^2 over 1024
// 15.9 / 12.1, 15.5 / 11.2 (wgrad 17.9 / 19.0), 1024^2 over 512 10.4 / 9.3, 9.7 / 8.8 (12.3 / 15.5), 512x1024 over 1024 as wgrad 17.5 / 13.4.
// A reduction of 8 or 16 is up to 0.4 us longer on them in dgrad and wgrad (128x128 over 16 3.8 / 4.0, 3.6 / 4.1).
inline bool dg_cut_sooner(int op, int64_t M, int64_t N, int64_t K) {
  const int64_t t7 = ((M + 127) / 128) * ((N + 127) / 128);
  if (t7 <= 18) return true;
  if (t7 <= 32) return op == GEMM_FWD || K >= (op == GEMM_WGRAD ? 2048 : 1024);
  return t7 <= 64 && K >= (op == GEMM_WGRAD ? 4096 : 1536);
}

// The library's choice for one product (0: the kernels of gemm_cut.h).  On top of the tile size and its kernel configuration:
// two 128x128 workgroups on a CU are bound by the CU's path from L2 (64 B per clock), so forward
// and dgrad products may run on 128x256 (else 256x128) tiles of 4 waves instead, one per CU: a pair
// of tiles that shares one operand panel through LDS, a quarter less L2->LDS traffic.  (The 0.92 below was
// measured with the eight-wave, two-stage form of these tiles; the present one, configurations 20 and 21,
// is 4-17 % faster still, so the rule may take them too seldom.)  The merged tiles come in whole rounds of one per CU.  A 128x128 workgroup alone
// on a CU runs at nearly twice the speed (0.55 of a full round's time for a product of at most 256
// tiles), one CU holding two makes the round a full one, and beyond 512 tiles the slots refill as
// they drain; in units of one full round of 512 tiles the two cost 0.55 / 1 / (tiles / 512) and
// 0.92 * ceil(tiles / 2 / 256).
inline int dg_pick(int op, int64_t M, int64_t N, int64_t K, int64_t lda, int64_t ldb) {
  if (dg_flavours().small[op] && dg_cut_sooner(op, M, N, K)) return 0;   // (a named 128x128 configuration is what runs)
  const int tile = dg_choose_variant(M, N, K, lda, ldb);
  if (tile == 7 && op != GEMM_WGRAD && dg_flavours().pair128) {
    const int64_t t = (M / 128) * (N / 128);
    const int wide = dg_shape_ok(20, M, N, K, lda, ldb) ? 20 : (dg_shape_ok(21, M, N, K, lda, ldb) ? 21 : 0);
    if (wide != 0) {
      const double c128 = t <= 256 ? 0.55 : (t <= 512 ? 1.0 : (double)t / 512.0);
      const double cw = 0.92 * (double)((t / 2 + 255) / 256);
      if (cw < c128 - 0.01) return wide;
    }
  }
  return dg_flavour(tile, op);
}

// Whether a forward product that dg_pick gives to merged tiles (20) takes them 192 wide (24): where the 256-wide ones leave a quarter of the chip idle.  Per round of
// 256 workgroups they cost 0.75 of the area and 1.04 for the larger share of loads.
// Measured, 256 wide / 192 wide (us, operands out of cache): 2048x3072x3072 51 / 45, 2048x3072x12288 167 / 156, 1024x6144x2048 29.0 / 26.4,
// 4096x1536x1536 28.6 / 25.4; a stage of three such layers forward 3307 -> 3219.
inline bool dg_narrow(int64_t M, int64_t N) {
  if (M % 128 != 0 || N % 192 != 0) return false;
  const int64_t wide = (M / 128) * ((N + 255) / 256), narrow = (M / 128) * (N / 192);
  return 0.75 * 1.04 * (double)((narrow + 255) / 256) < (double)((wide + 255) / 256);
}

// Whether one weight gradient that dg_pick gives to 128x128 tiles because its sides are multiples of 128 but not of 256 takes the EDGE form of
// the 256x256 ones (23): by the same rounds as dg_choose_variant, 1.05 for EDGE.  From 600 tiles on (just above one round of 128x128
// the two are even) and from 512 on in K (shorter ones spend their time in the epilogue: 9984x1152 over 64 23.4 / 26.7).  Below 768 k a part of a round of
// 128x128 tiles, which refill, counts as that part and a half, not as a whole one: 8832x2944 (3.1 rounds) over 512 68 / 72, 5760x4480 (3.08) over 576 73 / 76.
// Measured, 128x128 / 256x256 (us): 1920x7680 over 512, 2048, 8192 45 / 40, 99 / 74, 357 / 213; 5760x1920 over 2048 74 / 65; 9984x1152 75 / 67;
// where 128x128 stay: 2944^2 over 1024 40 / 41, 4480^2 over 2048 118 / 129, 6016x2944 104 / 116, 1920^2 26 / 47.
inline bool dg_wgrad_wide(int64_t M, int64_t N, int64_t K) {
  if (dg_shape_ok(5, M, N, K, M, N) || !dg_shape_ok(23, M, N, K, M, N)) return false;
  const int64_t t5 = ((M + 255) / 256) * ((N + 255) / 256), t7 = (M / 128) * (N / 128);
  double rounds7 = (double)((t7 + 511) / 512);
  if (K < 768 && (double)t7 / 512.0 + 0.5 < rounds7) rounds7 = (double)t7 / 512.0 + 0.5;
  return K >= 512 && t7 >= 600 && (double)((t5 + 255) / 256) * 4.0 / 1.15 * 1.05 <= rounds7 * 2.0;
}

// The configuration that runs in place of dg_pick's `v`, which knows the tiles' rounds but neither the epilogue nor the reduction's length.
// Measured on the products of layers 768 to 5120 wide over 512 to 6144 tokens, operands out of cache (us, dg_pick's / this one's):
//   forward on the 192-wide merged tiles, where dg_narrow says so or, from 1536 k on, where they take the place of 128x128 tiles in up to three rounds
//     of which the last is 7/8 full: 2048x9216x3072 129 / 123, GeLU 2048x9216x2304 114 / 109, 6144x3072x1536 67.2 / 64.9; in six rounds 225 / 243; shorter
//     reductions (128x128 tiles / these) 6144x3072x512 30.0 / 32.8, GeLU 6144x3072x1024 52 / 55, residual 4096x4608x64 22 / 27;
//   forward on 256x256 where the others need many more rounds (a round costs 70 on those, 46 on merged tiles, 50 on 128x128, which refill):
//     4096x9216x3072 225 / 212, 4096x10240x2560 239 / 207, 2048x20480x5120 403 / 380; short reductions 6144x6144x1536 130 / 140;
//   merged tiles 256x128, not 128x256, for outputs clearly wider than tall, in whole groups of 8 tile rows: dgrad 1024x5120x15360 222 / 194,
//     GeLU' 512x15360x3840 72 / 65, forward 1024x6912x2304 38 / 35; dgrad 2048x4096x12288 182 / 186, forward 3072x7680x2560 108 / 116;
//   dgrad on 256x256 tiles of at most 200 workgroups on four waves, not eight: 4096x2560x10240 224 / 200, 2048x5120x5120 117 / 107, GeLU'
//     1024x12288x3072 81 / 78; 240 and 256 workgroups are even, and so are 3072x3072x3072, 4096x2304x2304; GeLU' 4096x3072x768 9 % slower;
//   the ragged form of the 256x256 tiles for sides that are odd multiples of 128, where its rounds cost less (70 each, against 48 of 128x128 tiles
//     however those are merged, 42 under GeLU', whose epilogue is the longer one there; a single round against more than 1.2): forward 1920x7680x1920
//     80 / 53, 4224x3712x3712 129 / 100, 2048x5760x1920 54 / 50, 4480x6912x2304 179 / 130, 6016x4224x1408 94 / 71; dgrad 1408x10752x3584 137 / 96,
//     GeLU' 143 / 109; not 4096x5760x1920 91 / 97 (2.81 rounds of 128x128), 3200x4992x1664 63 / 76 (1.90), GeLU' 2944x9216x2304 138 / 143 (3.23).  Merged tiles that
//     nearly fill three rounds cost less than two of these, except 128x256 ones on a wide output: not 2304x10880x1792 residual 102 / 114 (2.99 of 3 rounds),
//     3072x8064x2688 127 / 133, GeLU 19328x1280x3008 143 / 160, 12800x1920x3200 159 / 170; but GeLU 1920x12800x3200 202 / 159 (2.93), and six against four
//     8832x5632x1472 168 / 152, dgrad 11776x4224x1152 141 / 126 (GeLU 13312x3712x1536 164 / 172).
inline int dg_at_launch(int v, int op, int mode, int64_t M, int64_t N, int64_t K, int64_t lda, int64_t ldb) {
  const int64_t t5 = ((M + 255) / 256) * ((N + 255) / 256), rounds5 = (t5 + 255) / 256;
  if ((v == 19 || v == 20 || v == 21) && op != GEMM_WGRAD && !dg_flavours().named && K >= 1024 && !dg_shape_ok(5, M, N, K, lda, ldb) &&
      dg_shape_ok(23, M, N, K, lda, ldb)) {
    const int64_t t7 = (M / 128) * (N / 128);
    const double f7 = (double)t7 / 512.0;
    const bool merged = rounds5 == 2 && (t7 + 511) / 512 == 3 && (v == 21 || (v == 20 && 2 * N < 3 * M));
    if (!merged && (70.0 * (double)rounds5 <= (mode == EPI_DGELU ? 42.0 : 48.0) * f7 || (rounds5 == 1 && mode != EPI_DGELU && f7 > 1.2))) return 23;
  }
  if (v == 20 && op == GEMM_FWD && dg_narrow(M, N)) return 24;
  if (dg_flavours().named) return v;
  if (op == GEMM_WGRAD) return v == 19 && mode == EPI_ACCUM_F32 && dg_wgrad_wide(M, N, K) ? 23 : v;
  if (v == 18 && op == GEMM_DGRAD) return t5 <= 200 && K >= (mode == EPI_DGELU ? 2304 : 3584) ? 17 : v;
  if (v != 19 && v != 20) return v;
  const int64_t t7 = (M / 128) * (N / 128), rounds_wide = (t7 / 2 + 255) / 256;
  if (op == GEMM_FWD && t5 > 256 && K >= 2304 && dg_shape_ok(17, M, N, K, lda, ldb) &&
      70.0 * (double)rounds5 < 0.97 * (v == 20 ? 46.0 * (double)rounds_wide : 50.0 * (double)t7 / 512.0)) return 17;
  if (v == 19) {
    if (op != GEMM_FWD || !dg_shape_ok(24, M, N, K, lda, ldb)) return v;
    const int64_t t24 = (M / 128) * (N / 192);
    return K >= 1536 && t24 >= 384 && t24 <= 768 && ((t24 + 255) / 256 * 256 - t24) * 8 <= 256 ? 24 : v;
  }
  const bool wide = mode == EPI_BIAS || mode == EPI_BIAS_GELU || mode == EPI_DGELU ? 2 * N >= 3 * M : N >= 3 * M;
  return wide && (M <= 2048 || M % 2048 == 0) && dg_shape_ok(21, M, N, K, lda, ldb) ? 21 : v;
}

// Split-K for weight-gradient GEMMs whose output has too few tiles to fill the chip: the
// reduction is cut into `splits` equal parts, each workgroup row of the grid writes its
// partial tile (EPI_STORE_F32) and splitk_reduce adds the partials to the accumulator in a
// fixed order, so the result stays run-to-run deterministic.  Returns 1 when no split pays.
inline int dg_wgrad_splits(int64_t M, int64_t N, int64_t K) {
  const int v = dg_choose_variant(M, N, K, M, N);
  GemmTile t;
  if (v == 0 || !dg_variant_tile(v, &t)) return 1;
  const int64_t tiles = ((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn), slots = t.bm == 256 ? 256 : 512;
  const int64_t nk = (K + DG_BK - 1) / DG_BK;
  int64_t s = slots / tiles;
  if (s > 8) s = 8;
  // plain tiles take equal parts only; the EDGE form's may differ by a k-tile
  while (s > 1 && ((v < 22 && nk % s != 0) || nk / s < 8)) --s;
  return (int)(s < 1 ? 1 : s);
}

// Whether `n` weight gradients over K (all four of a layer, of several layers) run as one launch, and on which kernel
// configuration (18, 19, 22, 23; 0: one by one).  In units of a full-chip round of 128x128 tiles a group takes its tiles / 512,
// or the whole rounds of 256x256 tiles its tiles need; one by one every product rounds up by itself.  With fewer tiles than
// slots cutting the reductions (dg_wgrad_splits) fills the chip better.  A group of 4096 and more 256x256 tiles whose matrices
// all prefer them alone stays one by one: at 8192 wide every matrix is whole rounds by itself and the group gains nothing; at
// widths where they are not (5120: 6.25, 6.25, 1.56 and 4.69 rounds) it would save a round or two, which is not taken.
// On 128x128 tiles over more than 8192 tokens the mixture of matrices costs more of the L2 than the last rounds give.
// Measured, one by one with their split sums / one launch, us of all weight gradients (4096 tokens unless given): one layer
// 1024 wide 197 / 126, 1920 wide 526 / 413, four layers of them 821 / 388 and 2063 / 1714, one and four layers 3072 wide over
// 2048 tokens 594 / 512 and 2358 / 1853; of 530 groups 576 to 7168 wide, 1 to 4 layers, 512 to 32768 tokens, none is more than 2 %
// slower than one by one.  Whole steps with 8 stacked micro-batches (TFLOP/s): 1024 wide 624 / 642 and 3072 wide 833 / 887, both
// on 256x256 tiles; 1920 wide over 32768 tokens on 128x128 tiles 806 / 758.
// (Measured while the += still stored 32-byte pieces; the larger tiles have gained more since: dg_group_wide.)
inline int dg_group_choice(const DgJob* jobs, int n, int64_t K) {
  if (!dg_flavours().group) return 0;   // a named weight-gradient configuration runs one by one
  int64_t t5 = 0, t7 = 0;
  bool plain5 = true, plain7 = true, edge = true, big_alone = true;
  for (int i = 0; i < n; ++i) {
    const int64_t M = jobs[i].M, N = jobs[i].N;
    const int alone = dg_choose_variant(M, N, K, M, N);
    big_alone = big_alone && (alone == 5 || alone == 23);
    plain5 = plain5 && dg_shape_ok(5, M, N, K, M, N);
    plain7 = plain7 && dg_shape_ok(7, M, N, K, M, N);
    edge = edge && dg_shape_ok(22, M, N, K, M, N);
    t5 += ((M + 255) / 256) * ((N + 255) / 256);
    t7 += ((M + 127) / 128) * ((N + 127) / 128);
  }
  if (t7 < 512 || !(plain7 || edge)) return 0;
  const double cost7 = (double)t7 / 512.0 + 0.2;
  const double cost5 = (double)((t5 + 255) / 256) * 2.0 / 1.15 * (plain5 ? 1.0 : 1.05);
  if (big_alone && t5 >= 16 * 256) return 0;
  if (cost5 <= cost7 && (plain5 || edge)) return plain5 ? 18 : 23;
  if (K > 8192) return 0;
  return plain7 ? 19 : 22;
}
// Whether a group that dg_group_choice gives to 128x128 tiles takes 256x256 ones after all (18; 23 where some matrix is no multiple of them).  In us
// per 1024 tokens and round: 256x256 tiles take 24 in whole rounds and 25 of epilogue per round's worth of tiles, 128x128 tiles 15 and
// 10 and refill as they drain, 0.3 of a round lost at the end (fitted over 512 and more tiles; off by up to 7 %, below 2048 tokens by more).
// Measured, 128x128 / 256x256 (us, all weight gradients): one layer 1920 wide over 4096 tokens 393 / 362, two 793 / 700, 1024 wide over 4096
// 137 / 121, 1536 wide 261 / 231; where 128x128 stay: 1600 wide, two layers over 2000 313 / 317, 4096 wide over 1024 581 / 625 (and, 2 % below
// the line by the estimate, 1280 wide, two layers over 8192 711 / 629).
inline int dg_group_wide(int variant, const DgJob* jobs, int n, int64_t K) {
  if ((variant != 19 && variant != 22) || K < 2048 || dg_flavours().named) return variant;
  int64_t t5 = 0, t7 = 0;
  bool plain = true, edge = true;
  for (int i = 0; i < n; ++i) {
    const int64_t M = jobs[i].M, N = jobs[i].N;
    plain = plain && dg_shape_ok(18, M, N, K, M, N);
    edge = edge && dg_shape_ok(23, M, N, K, M, N);
    t5 += ((M + 255) / 256) * ((N + 255) / 256);
    t7 += ((M + 127) / 128) * ((N + 127) / 128);
  }
  const double k = (double)K / 1024.0;
  const double us256 = 25.0 * (double)t5 / 256.0 + 24.0 * k * (double)((t5 + 255) / 256);
  const double us128 = ((double)t7 / 512.0 + 0.3) * (10.0 + 15.0 * k);
  if (!(plain || edge) || us256 > 0.97 * us128) return variant;
  return plain ? 18 : 23;
}
hipError_t launch_gemm_group(int variant, const DgJob* jobs, int n, int64_t K, hipStream_t st);   // gemm_wgrad.hip

// The launches, one translation unit per product; variant as above.
hipError_t launch_gemm_dma_fwd(int mode, int variant, const bf16* a, int64_t lda, const bf16* b, int64_t ldb, int64_t M, int64_t N,
                                 int64_t K, const EpiArgs<bf16>& epi, hipStream_t st);
hipError_t launch_gemm_dma_dgrad(int mode, int variant, const bf16* a, int64_t lda, const bf16* b, int64_t ldb, int64_t M, int64_t N,
                                 int64_t K, const EpiArgs<bf16>& epi, hipStream_t st);
hipError_t launch_gemm_dma_wgrad(int mode, int variant, const bf16* a, int64_t lda, const bf16* b, int64_t ldb, int64_t M, int64_t N,
                                 int64_t K, const EpiArgs<bf16>& epi, hipStream_t st, int splits);
// out[n] += the partial results of `splits` splits, in a fixed order (gemm_wgrad.hip)
hipError_t launch_splitk_reduce(const float* partial, int splits, int64_t n, float* out, hipStream_t st);

inline hipError_t launch_gemm_dma(int op, int mode, int variant, const bf16* a, int64_t lda, const bf16* b, int64_t ldb, int64_t M,
                                  int64_t N, int64_t K, const EpiArgs<bf16>& epi, hipStream_t st, int splits = 1) {
  if (op != GEMM_WGRAD && splits != 1) return hipErrorInvalidValue;
  if (op == GEMM_FWD) return launch_gemm_dma_fwd(mode, variant, a, lda, b, ldb, M, N, K, epi, st);
  if (op == GEMM_DGRAD) return launch_gemm_dma_dgrad(mode, variant, a, lda, b, ldb, M, N, K, epi, st);
  return launch_gemm_dma_wgrad(mode, variant, a, lda, b, ldb, M, N, K, epi, st, splits);
}

}  // namespace varuna
