// LayerNorm forward/backward (one wavefront per row, shuffle reductions) and
// deterministic two-stage column reductions for bias / gamma / beta gradients.
// All of these are HBM-bound: the arithmetic is fp32, the traffic is what counts.
#pragma once
#include <initializer_list>

#include "common.h"

namespace varuna {

constexpr int LN_ROWS_PER_BLOCK = 4;  // 4 waves, one row each
constexpr int CR_COLS = 64;           // columns per block in the column reductions
constexpr int CR_ROWLANES = 4;
constexpr int CR_CHUNK = 256;         // rows per partial

template <typename T, int VEC> struct VecLoad;
template <typename T> struct VecLoad<T, 1> {
  static __device__ __forceinline__ void load(const T* p, float* v) { v[0] = to_f32(p[0]); }
  static __device__ __forceinline__ void store(T* p, const float* v) { p[0] = from_f32<T>(v[0]); }
};
template <> struct VecLoad<float, 4> {
  static __device__ __forceinline__ void load(const float* p, float* v) {
    floatx4 t = *reinterpret_cast<const floatx4*>(p);
    v[0] = t[0]; v[1] = t[1]; v[2] = t[2]; v[3] = t[3];
  }
  static __device__ __forceinline__ void store(float* p, const float* v) {
    floatx4 t = {v[0], v[1], v[2], v[3]};
    *reinterpret_cast<floatx4*>(p) = t;
  }
};
template <> struct VecLoad<bf16, 8> {
  static __device__ __forceinline__ void load(const bf16* p, float* v) {
    bf16x8 t = *reinterpret_cast<const bf16x8*>(p);
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = (float)t[i];
  }
  static __device__ __forceinline__ void store(bf16* p, const float* v) {
    bf16x8 t;
#pragma unroll
    for (int i = 0; i < 8; ++i) t[i] = (bf16)v[i];
    *reinterpret_cast<bf16x8*>(p) = t;
  }
};

// y = gamma * (x - mean) * rstd + beta per row; biased variance, two passes
// (mean first, then centred second moment) so fp32 holds 1e-5 parity.
template <typename T, int VEC>
__global__ __launch_bounds__(LN_ROWS_PER_BLOCK* kWave) void layernorm_fwd_kernel(
    const T* __restrict__ x, const T* __restrict__ gamma, const T* __restrict__ beta,
    T* __restrict__ y, float* __restrict__ stats, int64_t rows, int h, float eps) {
  const int lane = threadIdx.x % kWave;
  const int64_t row = (int64_t)blockIdx.x * LN_ROWS_PER_BLOCK + threadIdx.x / kWave;
  if (row >= rows) return;
  const T* xr = x + row * h;
  float v[VEC], s = 0.f;
  for (int j = lane * VEC; j < h; j += kWave * VEC) {
    VecLoad<T, VEC>::load(xr + j, v);
#pragma unroll
    for (int i = 0; i < VEC; ++i) s += v[i];
  }
  const float mean = wave_sum(s) / (float)h;
  s = 0.f;
  for (int j = lane * VEC; j < h; j += kWave * VEC) {
    VecLoad<T, VEC>::load(xr + j, v);
#pragma unroll
    for (int i = 0; i < VEC; ++i) { float c = v[i] - mean; s += c * c; }
  }
  const float rstd = 1.0f / sqrtf(wave_sum(s) / (float)h + eps);
  if (stats && lane == 0) { stats[row] = mean; stats[rows + row] = rstd; }
  T* yr = y + row * h;
  float g[VEC], b[VEC];
  for (int j = lane * VEC; j < h; j += kWave * VEC) {
    VecLoad<T, VEC>::load(xr + j, v);
    VecLoad<T, VEC>::load(gamma + j, g);
    VecLoad<T, VEC>::load(beta + j, b);
#pragma unroll
    for (int i = 0; i < VEC; ++i) v[i] = g[i] * ((v[i] - mean) * rstd) + b[i];
    VecLoad<T, VEC>::store(yr + j, v);
  }
}

// dx = res + rstd * (dxhat - mean_j dxhat - xhat * mean_j(dxhat * xhat)),
// dxhat = dy * gamma, xhat = (x - mean) * rstd from the stored statistics.
template <typename T, int VEC>
__global__ __launch_bounds__(LN_ROWS_PER_BLOCK* kWave) void layernorm_bwd_dx_kernel(
    const T* __restrict__ dy, const T* __restrict__ x, const float* __restrict__ stats,
    const T* __restrict__ gamma, const T* __restrict__ res, T* __restrict__ dx, int64_t rows,
    int h) {
  const int lane = threadIdx.x % kWave;
  const int64_t row = (int64_t)blockIdx.x * LN_ROWS_PER_BLOCK + threadIdx.x / kWave;
  if (row >= rows) return;
  const float mean = stats[row], rstd = stats[rows + row];
  const T* xr = x + row * h;
  const T* dyr = dy + row * h;
  float vx[VEC], vd[VEC], g[VEC], s1 = 0.f, s2 = 0.f;
  for (int j = lane * VEC; j < h; j += kWave * VEC) {
    VecLoad<T, VEC>::load(xr + j, vx);
    VecLoad<T, VEC>::load(dyr + j, vd);
    VecLoad<T, VEC>::load(gamma + j, g);
#pragma unroll
    for (int i = 0; i < VEC; ++i) {
      float dxh = vd[i] * g[i];
      s1 += dxh;
      s2 += dxh * ((vx[i] - mean) * rstd);
    }
  }
  const float m1 = wave_sum(s1) / (float)h, m2 = wave_sum(s2) / (float)h;
  const T* rr = res + row * h;
  T* dxr = dx + row * h;
  float vr[VEC];
  for (int j = lane * VEC; j < h; j += kWave * VEC) {
    VecLoad<T, VEC>::load(xr + j, vx);
    VecLoad<T, VEC>::load(dyr + j, vd);
    VecLoad<T, VEC>::load(gamma + j, g);
    VecLoad<T, VEC>::load(rr + j, vr);
#pragma unroll
    for (int i = 0; i < VEC; ++i) {
      float xh = (vx[i] - mean) * rstd;
      vr[i] = vr[i] + rstd * (vd[i] * g[i] - m1 - xh * m2);
    }
    VecLoad<T, VEC>::store(dxr + j, vr);
  }
}

// Raw 16-byte vectors of a row held in registers (NC per lane), so that every tensor is read
// from memory once: rows of up to NC * 64 * VEC elements.
template <typename T, int VEC> struct RawVec { typedef T type __attribute__((ext_vector_type(VEC))); };

// EARLY: gamma and beta are fetched with the row, on their way during the reductions; it pays with their registers.
// COPY: the rows are also stored as they are.
template <typename T, int VEC, int NC, bool EARLY, bool COPY>
__global__ __launch_bounds__(LN_ROWS_PER_BLOCK* kWave) void layernorm_fwd_cached_kernel(
    const T* __restrict__ x, const T* __restrict__ gamma, const T* __restrict__ beta,
    T* __restrict__ y, float* __restrict__ stats, T* __restrict__ copy, int64_t rows, int h, float eps) {
  typedef typename RawVec<T, VEC>::type Raw;
  const int lane = threadIdx.x % kWave;
  const int64_t row = (int64_t)blockIdx.x * LN_ROWS_PER_BLOCK + threadIdx.x / kWave;
  if (row >= rows) return;
  const T* xr = x + row * h;
  Raw xc[NC], gc[EARLY ? NC : 1], bc[EARLY ? NC : 1];
  float s = 0.f;
  if constexpr (EARLY) {
#pragma unroll
    for (int it = 0; it < NC; ++it) {
      const int j = (it * kWave + lane) * VEC;
      if (j < h) {
        xc[it] = *reinterpret_cast<const Raw*>(xr + j);
        gc[it] = *reinterpret_cast<const Raw*>(gamma + j);
        bc[it] = *reinterpret_cast<const Raw*>(beta + j);
      }
    }
  }
#pragma unroll
  for (int it = 0; it < NC; ++it) {
    const int j = (it * kWave + lane) * VEC;
    if (j < h) {
      if constexpr (!EARLY) xc[it] = *reinterpret_cast<const Raw*>(xr + j);
      if constexpr (COPY) *reinterpret_cast<Raw*>(copy + row * h + j) = xc[it];
#pragma unroll
      for (int i = 0; i < VEC; ++i) s += to_f32(xc[it][i]);
    }
  }
  const float mean = wave_sum(s) / (float)h;
  s = 0.f;
#pragma unroll
  for (int it = 0; it < NC; ++it) {
    const int j = (it * kWave + lane) * VEC;
    if (j < h) {
#pragma unroll
      for (int i = 0; i < VEC; ++i) { const float c = to_f32(xc[it][i]) - mean; s += c * c; }
    }
  }
  const float rstd = 1.0f / sqrtf(wave_sum(s) / (float)h + eps);
  if (stats && lane == 0) { stats[row] = mean; stats[rows + row] = rstd; }
  T* yr = y + row * h;
#pragma unroll
  for (int it = 0; it < NC; ++it) {
    const int j = (it * kWave + lane) * VEC;
    if (j < h) {
      Raw g, b, o;
      if constexpr (EARLY) { g = gc[it]; b = bc[it]; }
      else { g = *reinterpret_cast<const Raw*>(gamma + j); b = *reinterpret_cast<const Raw*>(beta + j); }
#pragma unroll
      for (int i = 0; i < VEC; ++i) o[i] = from_f32<T>(to_f32(g[i]) * ((to_f32(xc[it][i]) - mean) * rstd) + to_f32(b[i]));
      *reinterpret_cast<Raw*>(yr + j) = o;
    }
  }
}

// (The residual row fetched ahead of the reductions as well was measured: 10.6 -> 13.6 us at 4096 x 1920.)
template <typename T, int VEC, int NC>
__device__ __forceinline__ void layernorm_bwd_dx_block(
    const T* __restrict__ dy, const T* __restrict__ x, const float* __restrict__ stats,
    const T* __restrict__ gamma, const T* __restrict__ res, T* __restrict__ dx, int64_t rows, int h, int64_t block) {
  typedef typename RawVec<T, VEC>::type Raw;
  const int lane = threadIdx.x % kWave;
  const int64_t row = block * LN_ROWS_PER_BLOCK + threadIdx.x / kWave;
  if (row >= rows) return;
  const float mean = stats[row], rstd = stats[rows + row];
  const T* xr = x + row * h;
  const T* dyr = dy + row * h;
  Raw xc[NC], dc[NC];   // the row of x and of dy; gamma is re-read (it stays in cache)
  float s1 = 0.f, s2 = 0.f;
#pragma unroll
  for (int it = 0; it < NC; ++it) {
    const int j = (it * kWave + lane) * VEC;
    if (j < h) {
      xc[it] = *reinterpret_cast<const Raw*>(xr + j);
      dc[it] = *reinterpret_cast<const Raw*>(dyr + j);
      const Raw g = *reinterpret_cast<const Raw*>(gamma + j);
#pragma unroll
      for (int i = 0; i < VEC; ++i) {
        const float dxh = to_f32(dc[it][i]) * to_f32(g[i]);
        s1 += dxh;
        s2 += dxh * ((to_f32(xc[it][i]) - mean) * rstd);
      }
    }
  }
  const float m1 = wave_sum(s1) / (float)h, m2 = wave_sum(s2) / (float)h;
  const T* rr = res + row * h;
  T* dxr = dx + row * h;
#pragma unroll
  for (int it = 0; it < NC; ++it) {
    const int j = (it * kWave + lane) * VEC;
    if (j < h) {
      const Raw g = *reinterpret_cast<const Raw*>(gamma + j), r = *reinterpret_cast<const Raw*>(rr + j);
      Raw o;
#pragma unroll
      for (int i = 0; i < VEC; ++i) {
        const float xh = (to_f32(xc[it][i]) - mean) * rstd;
        o[i] = from_f32<T>(to_f32(r[i]) + rstd * (to_f32(dc[it][i]) * to_f32(g[i]) - m1 - xh * m2));
      }
      *reinterpret_cast<Raw*>(dxr + j) = o;
    }
  }
}

template <typename T, int VEC, int NC>
__global__ __launch_bounds__(LN_ROWS_PER_BLOCK* kWave) void layernorm_bwd_dx_cached_kernel(
    const T* __restrict__ dy, const T* __restrict__ x, const float* __restrict__ stats,
    const T* __restrict__ gamma, const T* __restrict__ res, T* __restrict__ dx, int64_t rows, int h) {
  layernorm_bwd_dx_block<T, VEC, NC>(dy, x, stats, gamma, res, dx, rows, h, blockIdx.x);
}

// Stage 1 of a column reduction over rows [chunk*CR_CHUNK, +CR_CHUNK).
// LNMODE 0: partial[chunk][c] = sum_t a[t,c].
// LNMODE 1: partial[chunk][c] = sum_t a[t,c]*xhat[t,c] (dgamma) and
//           partial[chunk][n+c] = sum_t a[t,c] (dbeta), xhat from x and stats.
template <typename T, int LNMODE>
__global__ __launch_bounds__(CR_COLS* CR_ROWLANES) void colreduce_partial_kernel(
    const T* __restrict__ a, const T* __restrict__ x, const float* __restrict__ stats,
    float* __restrict__ partial, int64_t rows, int64_t n) {
  __shared__ float sh[2][CR_ROWLANES][CR_COLS];
  const int c = threadIdx.x % CR_COLS, rl = threadIdx.x / CR_COLS;
  const int64_t col = (int64_t)blockIdx.x * CR_COLS + c;
  const int64_t r0 = (int64_t)blockIdx.y * CR_CHUNK;
  const int64_t r1 = (r0 + CR_CHUNK < rows) ? r0 + CR_CHUNK : rows;
  float s0 = 0.f, s1 = 0.f;
  if (col < n) {
    for (int64_t t = r0 + rl; t < r1; t += CR_ROWLANES) {
      float v = to_f32(a[t * n + col]);
      if (LNMODE) {
        float xh = (to_f32(x[t * n + col]) - stats[t]) * stats[rows + t];
        s0 += v * xh;
        s1 += v;
      } else {
        s0 += v;
      }
    }
  }
  sh[0][rl][c] = s0;
  sh[1][rl][c] = s1;
  __syncthreads();
  if (rl == 0 && col < n) {
    float t0 = 0.f, t1 = 0.f;
#pragma unroll
    for (int i = 0; i < CR_ROWLANES; ++i) { t0 += sh[0][i][c]; t1 += sh[1][i][c]; }
    const int64_t width = LNMODE ? 2 * n : n;
    partial[(int64_t)blockIdx.y * width + col] = t0;
    if (LNMODE) partial[(int64_t)blockIdx.y * width + n + col] = t1;
  }
}

// Stage 2: out0[c] += sum_chunks partial[chunk][c]; with out1, also the second half.  Column c of the concatenation of both
// outputs per thread lane, the chunks over 8 groups of lanes (summed through LDS in a fixed order): the kernel lasts as
// long as one thread's serial loads.
constexpr int CF_COLS = 32, CF_LANES = 8;
template <int COLS, int LANES>
__device__ __forceinline__ void colreduce_final_block(const float* __restrict__ partial, int64_t pitch, int nchunks, int64_t n,
                                                      float* __restrict__ out0, float* __restrict__ out1, int64_t blk) {
  __shared__ float sh[LANES][COLS];
  const int c = threadIdx.x % COLS, l = threadIdx.x / COLS;
  const int64_t width = out1 ? 2 * n : n, col = blk * COLS + c;
  float t = 0.f;
  if (col < width)
#pragma unroll 4
    for (int k = l; k < nchunks; k += LANES) t += partial[(int64_t)k * pitch + col];
  if constexpr (LANES > 1) {
    sh[l][c] = t;
    __syncthreads();
    if (l != 0) return;
#pragma unroll
    for (int i = 1; i < LANES; ++i) t += sh[i][c];
  }
  if (col >= width) return;
  if (col < n) out0[col] += t; else out1[col - n] += t;
}
template <int COLS, int LANES>
__global__ __launch_bounds__(COLS* LANES) void colreduce_final_kernel(const float* __restrict__ partial, int nchunks, int64_t n,
                                                                      float* __restrict__ out0, float* __restrict__ out1) {
  colreduce_final_block<COLS, LANES>(partial, out1 ? 2 * n : n, nchunks, n, out0, out1, blockIdx.x);
}
inline void launch_colreduce_final(const float* partial, int nchunks, int64_t n, float* out0, float* out1, hipStream_t st) {
  const int64_t width = out1 ? 2 * n : n;
  if (nchunks <= CF_LANES / 2)   // a thread per column: no lanes to spare on so few chunks (1 x 2^20 sums 23.4 -> 13.9 us for both stages)
    hipLaunchKernelGGL((colreduce_final_kernel<256, 1>), dim3((unsigned)((width + 255) / 256)), dim3(256), 0, st, partial, nchunks, n, out0, out1);
  else
    hipLaunchKernelGGL((colreduce_final_kernel<CF_COLS, CF_LANES>), dim3((unsigned)((width + CF_COLS - 1) / CF_COLS)), dim3(CF_COLS * CF_LANES), 0, st, partial, nchunks, n, out0, out1);
}

template <typename T> constexpr int ln_vec() { return 16 / (int)sizeof(T); }
inline bool ln_aligned16(std::initializer_list<const void*> ps) {
  for (const void* p : ps)
    if (reinterpret_cast<uintptr_t>(p) & 15) return false;
  return true;
}

// copy (optional): a second place for the rows of x, read once for both; 4096 x 1920 in bf16 9.4 + 9.7 us as two launches.
template <typename T>
inline hipError_t launch_layernorm_fwd(const T* x, const T* gamma, const T* beta, T* y, float* stats,
                                       int64_t rows, int h, float eps, hipStream_t st, T* copy = nullptr) {
  dim3 grid((unsigned)((rows + LN_ROWS_PER_BLOCK - 1) / LN_ROWS_PER_BLOCK)), block(LN_ROWS_PER_BLOCK * kWave);
  constexpr int V = ln_vec<T>();
  const int nv = (h / V + kWave - 1) / kWave;  // 16-byte vectors per lane
  if (copy && !(h % V == 0 && nv <= 16 && ln_aligned16({x, gamma, beta, y, copy}))) {   // no kernel that holds the row
    const hipError_t e = hipMemcpyAsync(copy, x, (size_t)rows * h * sizeof(T), hipMemcpyDeviceToDevice, st);
    if (e != hipSuccess) return e;
    x = copy;
    copy = nullptr;
  }
  if (h % V == 0 && ln_aligned16({x, gamma, beta, y})) {
    // EARLY up to 8 vectors (beyond, registers run out), unless a row is one vector per lane (it then costs more waves than it
    // hides), or the rows are one round of the chip without it and two with it (5 to 8 vectors: 3 blocks of 4 rows per CU with
    // it, 5 in bf16 and 7 in fp32 without).  Measured, without / with (kernel us, row just written): bf16 512 x 4096 9.1 / 6.2,
    // 1000 x 1920 6.0 / 5.4, 16384 x 4096 48.0 / 42.7, but 16384 x 256 8.6 / 9.8, 4096 x 3072 11.7 / 12.4, fp32 4096 x 1536
    // 10.6 / 11.5.  (fp32 held to 128 registers for a fourth block spills: 16384 x 2048 49.0 / 58.8.)
    const bool early = nv >= 2 && !(nv > 4 && rows > 3072 && rows <= (sizeof(T) == 2 ? 5120 : 7168));
#define VARUNA_LNF(NC_, E_)                                                                                                             \
  do {                                                                                                                                  \
    if (copy) hipLaunchKernelGGL((layernorm_fwd_cached_kernel<T, V, NC_, E_, true>), grid, block, 0, st, x, gamma, beta, y, stats, copy, rows, h, eps); \
    else hipLaunchKernelGGL((layernorm_fwd_cached_kernel<T, V, NC_, E_, false>), grid, block, 0, st, x, gamma, beta, y, stats, copy, rows, h, eps);     \
  } while (0)
    if (nv <= 4) { if (early) VARUNA_LNF(4, true); else VARUNA_LNF(4, false); }
    else if (nv <= 8) { if (early) VARUNA_LNF(8, true); else VARUNA_LNF(8, false); }
    else if (nv <= 16) VARUNA_LNF(16, false);
#undef VARUNA_LNF
    else hipLaunchKernelGGL((layernorm_fwd_kernel<T, V>), grid, block, 0, st, x, gamma, beta, y, stats, rows, h, eps);
  } else
    hipLaunchKernelGGL((layernorm_fwd_kernel<T, 1>), grid, block, 0, st, x, gamma, beta, y, stats, rows, h, eps);
  return hipGetLastError();
}

// The same partial column sums with 16-byte accesses.  HBM-bound, so what counts is how many loads are in flight.  A block takes
// 8 column groups of VEC columns (128-byte row segments) x 32 row lanes, or 32 groups x 8 row lanes: a quarter of the blocks, for
// the same number of partials, with longer row segments.  The wide form serves what it fills the chip with (2 blocks per CU; 3
// for the gamma / beta sums, which read twice as much per block).  Measured, narrow / wide (us, both stages or the whole backward):
// sums in bf16 1024 x 32768 14.2 / 13.2, 16384 x 8192 44.5 / 41.4, fp32 512 x 32768 14.1 / 12.8, but 16384 x 256 fp32 backward
// 20.3 / 21.7; LayerNorm backward in bf16 4096 x 1920 20.9 / 36.4, 16384 x 1920 58.6 / 65.7, 16384 x 8192 360 / 338, fp32
// 4096 x 1024 19.2 / 23.5, 16384 x 8192 825 / 794.  Of few rows the narrow form leaves most row lanes idle: 1 x 2^20 23.3 / 17.7.
// Rows of 256 KB and more are taken one at a time, not four: fp32 512 x 131072 47.1 -> 39.8.
constexpr int CRV_CG = 8, CRV_RL = 32;   // column groups and row lanes of a block
template <typename T, int LNMODE, int VEC, int CG, int RL, int UNROLL = 4>
__device__ __forceinline__ void colreduce_partial_block(
    const T* __restrict__ a, const T* __restrict__ x, const float* __restrict__ stats, int64_t rows, int64_t n, int64_t colblk,
    int64_t chunk, float (&sh)[2][RL][CG * VEC + 4]) {
  const int cg = threadIdx.x % CG, rl = threadIdx.x / CG;
  const int64_t col = (colblk * CG + cg) * VEC;
  const int64_t r0 = chunk * CR_CHUNK;
  const int nr = (int)((rows - r0 < CR_CHUNK) ? rows - r0 : CR_CHUNK);
  float s0[VEC], s1[VEC];
#pragma unroll
  for (int i = 0; i < VEC; ++i) { s0[i] = 0.f; s1[i] = 0.f; }
  if (col < n) {
#pragma unroll UNROLL
    for (int t = rl; t < nr; t += RL) {
      float v[VEC];
      VecLoad<T, VEC>::load(a + (r0 + t) * n + col, v);
      if (LNMODE) {
        float xv[VEC];
        VecLoad<T, VEC>::load(x + (r0 + t) * n + col, xv);
        const float mu = stats[r0 + t], rs = stats[rows + r0 + t];
#pragma unroll
        for (int i = 0; i < VEC; ++i) { s0[i] += v[i] * ((xv[i] - mu) * rs); s1[i] += v[i]; }
      } else {
#pragma unroll
        for (int i = 0; i < VEC; ++i) s0[i] += v[i];
      }
    }
  }
#pragma unroll
  for (int i = 0; i < VEC; ++i) { sh[0][rl][cg * VEC + i] = s0[i]; if (LNMODE) sh[1][rl][cg * VEC + i] = s1[i]; }
  __syncthreads();
}
// Sum number c of the block (LNMODE: first the columns' dy * xhat, then their dy).
template <int COLS, int RL>
__device__ __forceinline__ float colreduce_block_sum(const float (&sh)[2][RL][COLS + 4], int which, int c) {
  float t = 0.f;
#pragma unroll
  for (int i = 0; i < RL; ++i) t += sh[which][i][c];
  return t;
}

template <typename T, int LNMODE, int VEC, int CG, int RL, int UNROLL>
__global__ __launch_bounds__(256) void colreduce_partial_vec_kernel(
    const T* __restrict__ a, const T* __restrict__ x, const float* __restrict__ stats,
    float* __restrict__ partial, int64_t rows, int64_t n) {
  constexpr int COLS = CG * VEC;
  __shared__ float sh[2][RL][COLS + 4];
  colreduce_partial_block<T, LNMODE, VEC, CG, RL, UNROLL>(a, x, stats, rows, n, blockIdx.x, blockIdx.y, sh);
  const int64_t width = LNMODE ? 2 * n : n;
  for (int t = threadIdx.x; t < (LNMODE ? 2 : 1) * COLS; t += 256) {
    const int which = t / COLS, c = t % COLS;
    const int64_t gc = (int64_t)blockIdx.x * COLS + c;
    if (gc < n) partial[(int64_t)blockIdx.y * width + which * n + gc] = colreduce_block_sum<COLS, RL>(sh, which, c);
  }
}

// All six column reductions of one layer's backward in one launch and their second stages in another: job j sums
// a[rows, n] (x == null) or is a LayerNorm's gamma / beta pair; it owns column blocks first[j] .. first[j+1]-1 of the
// first stage, final column blocks ffirst[j] .. of the second, and `width` columns of the partials from pcol[j] on (row
// pitch `pitch`).  With one chunk of rows the first stage adds to the outputs itself.
// Twelve launches of a layer become two, or one up to 256 tokens: tiny fp32 step (16 layer backwards) 1097 -> 940 us.
constexpr int kMaxReduceJobs = 6;
template <typename T>
struct ReduceJob { const T* a; const T* x; const float* stats; float* out0; float* out1; int n; };
template <typename T>
struct ReduceJobs {
  int n_jobs, nchunks;
  int64_t rows, pitch;
  int first[kMaxReduceJobs + 1], ffirst[kMaxReduceJobs + 1], pcol[kMaxReduceJobs];
  ReduceJob<T> job[kMaxReduceJobs];
};
template <typename T, int VEC>
__device__ __forceinline__ void colreduce_jobs_block(const ReduceJobs<T>& g, float* __restrict__ partial, int blk, int chunk) {
  constexpr int COLS = CRV_CG * VEC;
  __shared__ float sh[2][CRV_RL][COLS + 4];
  int j = 0;
  while (j + 1 < g.n_jobs && blk >= g.first[j + 1]) ++j;
  const ReduceJob<T> w = g.job[j];
  const int colblk = blk - g.first[j];
  const bool ln = w.x != nullptr;
  if (ln) colreduce_partial_block<T, 1, VEC, CRV_CG, CRV_RL>(w.a, w.x, w.stats, g.rows, w.n, colblk, chunk, sh);
  else colreduce_partial_block<T, 0, VEC, CRV_CG, CRV_RL>(w.a, nullptr, nullptr, g.rows, w.n, colblk, chunk, sh);
  if ((int)threadIdx.x >= (ln ? 2 : 1) * COLS) return;
  const int which = threadIdx.x / COLS, c = threadIdx.x % COLS;
  const int64_t gc = (int64_t)colblk * COLS + c;
  if (gc >= w.n) return;
  const float t = colreduce_block_sum<COLS, CRV_RL>(sh, which, c);
  if (g.nchunks == 1) (which ? w.out1 : w.out0)[gc] += t;
  else partial[(int64_t)chunk * g.pitch + g.pcol[j] + which * w.n + gc] = t;
}
template <typename T, int VEC>
__global__ __launch_bounds__(256) void colreduce_jobs_partial_kernel(ReduceJobs<T> g, float* __restrict__ partial) {
  colreduce_jobs_block<T, VEC>(g, partial, blockIdx.x, blockIdx.y);
}

// The first stage of some column reductions and a LayerNorm backward's dx in one launch: neither reads what the other writes, each alone
// is a launch of a few microseconds that hardly fills the chip, and for the LayerNorm's own gamma / beta sums both read the same rows.
// The reductions' blocks (the longer ones) come first.
template <typename T>
struct LnBwdDx { const T* dy; const T* x; const float* stats; const T* gamma; const T* res; T* dx; int64_t rows; int h; };
template <typename T, int VEC, int NC>
__global__ __launch_bounds__(256) void layernorm_bwd_jobs_kernel(LnBwdDx<T> d, ReduceJobs<T> g, float* __restrict__ partial) {
  static_assert(LN_ROWS_PER_BLOCK * kWave == 256, "one block size for both");
  const int per = g.first[g.n_jobs];
  const int64_t dx_block = (int64_t)blockIdx.x - (int64_t)per * g.nchunks;
  if (dx_block < 0) colreduce_jobs_block<T, VEC>(g, partial, (int)(blockIdx.x % per), (int)(blockIdx.x / per));
  else layernorm_bwd_dx_block<T, VEC, NC>(d.dy, d.x, d.stats, d.gamma, d.res, d.dx, d.rows, d.h, dx_block);
}
template <typename T>
__global__ __launch_bounds__(CF_COLS* CF_LANES) void colreduce_jobs_final_kernel(ReduceJobs<T> g, const float* __restrict__ partial) {
  int j = 0;
  while (j + 1 < g.n_jobs && (int)blockIdx.x >= g.ffirst[j + 1]) ++j;
  const ReduceJob<T> w = g.job[j];
  colreduce_final_block<CF_COLS, CF_LANES>(partial + g.pcol[j], g.pitch, g.nchunks, w.n, w.out0, w.out1, (int64_t)((int)blockIdx.x - g.ffirst[j]));
}

template <typename T, int LNMODE>
inline void launch_colreduce_partial(const T* a, const T* x, const float* stats, float* partial, int64_t rows, int64_t n,
                                     hipStream_t st) {
  const int nch = (int)((rows + CR_CHUNK - 1) / CR_CHUNK);
  constexpr int VEC = 16 / sizeof(T);
  const bool aligned = (reinterpret_cast<uintptr_t>(a) % 16 == 0) && (x == nullptr || reinterpret_cast<uintptr_t>(x) % 16 == 0);
  if (n % VEC == 0 && aligned) {
    const int64_t wide = (n + CRV_RL * VEC - 1) / (CRV_RL * VEC);
    if (wide * nch >= (LNMODE ? 768 : 512)) {
      dim3 g((unsigned)wide, (unsigned)nch);
      if (n * (int64_t)sizeof(T) >= (1 << 18)) hipLaunchKernelGGL((colreduce_partial_vec_kernel<T, LNMODE, VEC, CRV_RL, CRV_CG, 1>), g, dim3(256), 0, st, a, x, stats, partial, rows, n);
      else hipLaunchKernelGGL((colreduce_partial_vec_kernel<T, LNMODE, VEC, CRV_RL, CRV_CG, 4>), g, dim3(256), 0, st, a, x, stats, partial, rows, n);
    } else {
      dim3 g((unsigned)((n + CRV_CG * VEC - 1) / (CRV_CG * VEC)), (unsigned)nch);
      hipLaunchKernelGGL((colreduce_partial_vec_kernel<T, LNMODE, VEC, CRV_CG, CRV_RL, 4>), g, dim3(256), 0, st, a, x, stats, partial, rows, n);
    }
  } else {
    dim3 g((unsigned)((n + CR_COLS - 1) / CR_COLS), (unsigned)nch);
    hipLaunchKernelGGL((colreduce_partial_kernel<T, LNMODE>), g, dim3(CR_COLS * CR_ROWLANES), 0, st, a, x, stats, partial, rows, n);
  }
}

inline int colreduce_chunks(int64_t rows) { return (int)((rows + CR_CHUNK - 1) / CR_CHUNK); }

// dx = res + LN'(dy) alone (one launch).
template <typename T>
inline hipError_t launch_layernorm_bwd_dx(const T* dy, const T* x, const float* stats, const T* gamma,
                                          const T* res, T* dx, int64_t rows, int h, hipStream_t st) {
  dim3 grid((unsigned)((rows + LN_ROWS_PER_BLOCK - 1) / LN_ROWS_PER_BLOCK)), block(LN_ROWS_PER_BLOCK * kWave);
  constexpr int V = ln_vec<T>();
  if (h % V == 0 && ln_aligned16({dy, x, gamma, res, dx})) {
    const int nv = (h / V + kWave - 1) / kWave;
    if (nv <= 4) hipLaunchKernelGGL((layernorm_bwd_dx_cached_kernel<T, V, 4>), grid, block, 0, st, dy, x, stats, gamma, res, dx, rows, h);
    else if (nv <= 8) hipLaunchKernelGGL((layernorm_bwd_dx_cached_kernel<T, V, 8>), grid, block, 0, st, dy, x, stats, gamma, res, dx, rows, h);
    else if (nv <= 16) hipLaunchKernelGGL((layernorm_bwd_dx_cached_kernel<T, V, 16>), grid, block, 0, st, dy, x, stats, gamma, res, dx, rows, h);
    else hipLaunchKernelGGL((layernorm_bwd_dx_kernel<T, V>), grid, block, 0, st, dy, x, stats, gamma, res, dx, rows, h);
  } else
    hipLaunchKernelGGL((layernorm_bwd_dx_kernel<T, 1>), grid, block, 0, st, dy, x, stats, gamma, res, dx, rows, h);
  return hipGetLastError();
}

// dgamma += sum_t dy * xhat, dbeta += sum_t dy (two launches; they read dy, x and the statistics only,
// so they need not run on the stream that carries dx).
template <typename T>
inline hipError_t launch_layernorm_bwd_params(const T* dy, const T* x, const float* stats, float* dgamma, float* dbeta,
                                              float* partial, int64_t rows, int h, hipStream_t st) {
  const int nch = colreduce_chunks(rows);
  launch_colreduce_partial<T, 1>(dy, x, stats, partial, rows, (int64_t)h, st);
  launch_colreduce_final(partial, nch, (int64_t)h, dgamma, dbeta, st);
  return hipGetLastError();
}

template <typename T>
inline hipError_t launch_colsum(const T* a, float* out, float* partial, int64_t rows, int64_t n, hipStream_t st) {
  const int nch = colreduce_chunks(rows);
  launch_colreduce_partial<T, 0>(a, (const T*)nullptr, (const float*)nullptr, partial, rows, n, st);
  launch_colreduce_final(partial, nch, n, out, nullptr, st);
  return hipGetLastError();
}

// The job table of some column reductions over the same rows; false where their columns are no whole 16-byte pieces.
template <typename T>
inline bool make_reduce_jobs(ReduceJobs<T>* out, const ReduceJob<T>* jobs, int n_jobs, int64_t rows) {
  constexpr int VEC = 16 / sizeof(T);
  for (int i = 0; i < n_jobs; ++i)
    if (jobs[i].n % VEC != 0 || !ln_aligned16({jobs[i].a, jobs[i].x})) return false;
  ReduceJobs<T>& g = *out;
  g = ReduceJobs<T>{};
  g.n_jobs = n_jobs; g.nchunks = colreduce_chunks(rows); g.rows = rows;
  int64_t pitch = 0;
  for (int i = 0; i < n_jobs; ++i) {
    const int width = (jobs[i].x ? 2 : 1) * jobs[i].n;
    g.job[i] = jobs[i];
    g.pcol[i] = (int)pitch;
    g.first[i + 1] = g.first[i] + (jobs[i].n + CRV_CG * VEC - 1) / (CRV_CG * VEC);
    g.ffirst[i + 1] = g.ffirst[i] + (width + CF_COLS - 1) / CF_COLS;
    pitch += width;
  }
  g.pitch = pitch;
  return true;
}
template <typename T>
inline void launch_reduce_jobs_final(const ReduceJobs<T>& g, const float* partial, hipStream_t st) {
  if (g.nchunks > 1) hipLaunchKernelGGL((colreduce_jobs_final_kernel<T>), dim3((unsigned)g.ffirst[g.n_jobs]), dim3(CF_COLS * CF_LANES), 0, st, g, partial);
}

// The jobs of one layer; partial: (sum of the jobs' widths) * colreduce_chunks(rows) floats.
template <typename T>
inline hipError_t launch_reduce_jobs(const ReduceJob<T>* jobs, int n_jobs, float* partial, int64_t rows, hipStream_t st) {
  ReduceJobs<T> g;
  if (!make_reduce_jobs<T>(&g, jobs, n_jobs, rows)) {   // one by one
    for (int i = 0; i < n_jobs; ++i) {
      const ReduceJob<T>& w = jobs[i];
      const hipError_t e = w.x ? launch_layernorm_bwd_params<T>(w.a, w.x, w.stats, w.out0, w.out1, partial, rows, w.n, st)
                               : launch_colsum<T>(w.a, w.out0, partial, rows, w.n, st);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  hipLaunchKernelGGL((colreduce_jobs_partial_kernel<T, 16 / (int)sizeof(T)>), dim3((unsigned)g.first[n_jobs], (unsigned)g.nchunks), dim3(256), 0, st, g, partial);
  launch_reduce_jobs_final<T>(g, partial, st);
  return hipGetLastError();
}

// dx of a LayerNorm and some column reductions over the same rows: the dx and the reductions' first stage share a launch up to eight vectors
// per lane, the rows that the joint kernel holds; where both are long it costs nothing (micro-batches of a stage, two launches / one: bf16
// 16384 x 2048 3807 / 3811, 16384 x 4096 11479 / 11454, 65536 x 1024 5453 / 5443, fp32 8192 x 1024 5157 / 5125).  Three launches become two, or one up to 256 rows; measured for a LayerNorm alone (us): bf16 64x64 13.2 -> 8.6, 512x768 13.6 -> 11.0,
// 1000x4096 19.9 -> 14.0, 4096x1920 20.9 -> 18.3, 16384x256 18.2 -> 12.4, 16384x1920 60.4 -> 58.8; fp32 64x64 13.7 -> 8.5, 4096x1024
// 19.4 -> 18.7.
template <typename T>
inline hipError_t launch_layernorm_bwd_jobs(const LnBwdDx<T>& d, const ReduceJob<T>* jobs, int n_jobs, float* partial, hipStream_t st) {
  constexpr int V = ln_vec<T>();
  ReduceJobs<T> g;
  const int nv = (d.h / V + kWave - 1) / kWave;
  const int64_t dx_blocks = (d.rows + LN_ROWS_PER_BLOCK - 1) / LN_ROWS_PER_BLOCK;
  if (d.h % V == 0 && ln_aligned16({d.dy, d.x, d.gamma, d.res, d.dx}) && nv <= 8 && d.rows <= (1 << 20) && make_reduce_jobs<T>(&g, jobs, n_jobs, d.rows)) {
    const dim3 grid((unsigned)(dx_blocks + (int64_t)g.first[n_jobs] * g.nchunks)), block(256);
    if (nv <= 4) hipLaunchKernelGGL((layernorm_bwd_jobs_kernel<T, V, 4>), grid, block, 0, st, d, g, partial);
    else hipLaunchKernelGGL((layernorm_bwd_jobs_kernel<T, V, 8>), grid, block, 0, st, d, g, partial);
    launch_reduce_jobs_final<T>(g, partial, st);
    return hipGetLastError();
  }
  const hipError_t e = launch_layernorm_bwd_dx<T>(d.dy, d.x, d.stats, d.gamma, d.res, d.dx, d.rows, d.h, st);
  return e != hipSuccess ? e : launch_reduce_jobs<T>(jobs, n_jobs, partial, d.rows, st);
}

// dx plus the gamma / beta gradient accumulation.
template <typename T>
inline hipError_t launch_layernorm_bwd(const T* dy, const T* x, const float* stats, const T* gamma,
                                       const T* res, T* dx, float* dgamma, float* dbeta,
                                       float* partial, int64_t rows, int h, hipStream_t st) {
  // (the wide form of the partial sums fills the chip by itself; longer rows than 8 vectors per lane have no joint kernel)
  constexpr int V = ln_vec<T>();
  if (h <= 8 * kWave * V && (int64_t)((h + CRV_RL * V - 1) / (CRV_RL * V)) * colreduce_chunks(rows) < 768) {
    const ReduceJob<T> job{dy, x, stats, dgamma, dbeta, h};
    return launch_layernorm_bwd_jobs<T>({dy, x, stats, gamma, res, dx, rows, h}, &job, 1, partial, st);
  }
  hipError_t e = launch_layernorm_bwd_dx<T>(dy, x, stats, gamma, res, dx, rows, h, st);
  if (e != hipSuccess) return e;
  return launch_layernorm_bwd_params<T>(dy, x, stats, dgamma, dbeta, partial, rows, h, st);
}

// out = dropout(in) with the mask of one site (backward of a residual-branch dropout: the
// gradient that enters the branch's GEMMs and bias reduction).  A thread takes 4 rows x 8 columns, two mask patches: one
// generator call per 16 elements (a thread per row of a patch made one per 4, which bound the kernel) and 16-byte (fp32:
// two 16-byte) accesses.  4096 x 1024 in bf16: 9.6 -> 5.8 us.
template <typename T, bool VEC>
__global__ __launch_bounds__(256) void dropout_apply_kernel(const T* __restrict__ in, T* __restrict__ out, int64_t rows,
                                                            int64_t cols, DropArgs drop) {
  typedef T Tx8 __attribute__((ext_vector_type(8)));
  const int64_t cpr = (cols + 7) / 8, total = (rows + 3) / 4 * cpr;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t rp = i / cpr, c0 = (i % cpr) * 8;
    uint32_t w[2][4];
    drop_patch(drop, (uint32_t)rp, (uint32_t)(c0 >> 2), w[0]);
    drop_patch(drop, (uint32_t)rp, (uint32_t)(c0 >> 2) + 1, w[1]);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if (rp * 4 + r >= rows) break;
      const int64_t base = (rp * 4 + r) * cols + c0;
      if constexpr (VEC) {
        Tx8 v = *reinterpret_cast<const Tx8*>(in + base);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = drop_keep(drop, w[e >> 2][r], e & 3) ? from_f32<T>(to_f32((T)v[e]) * drop.scale) : from_f32<T>(0.f);
        *reinterpret_cast<Tx8*>(out + base) = v;
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (c0 + e < cols) out[base + e] = drop_keep(drop, w[e >> 2][r], e & 3) ? from_f32<T>(to_f32(in[base + e]) * drop.scale) : from_f32<T>(0.f);
      }
    }
  }
}

template <typename T>
inline hipError_t launch_dropout_apply(const T* in, T* out, int64_t rows, int64_t cols, const DropArgs& drop, hipStream_t st) {
  const int64_t total = (rows + 3) / 4 * ((cols + 7) / 8);
  int64_t nblk = (total + 255) / 256;
  if (nblk > 16384) nblk = 16384;
  if (nblk < 1) nblk = 1;
  const uintptr_t align = 8 * sizeof(T) - 1;
  if (cols % 8 == 0 && ((reinterpret_cast<uintptr_t>(in) | reinterpret_cast<uintptr_t>(out)) & align) == 0)
    hipLaunchKernelGGL((dropout_apply_kernel<T, true>), dim3((unsigned)nblk), dim3(256), 0, st, in, out, rows, cols, drop);
  else hipLaunchKernelGGL((dropout_apply_kernel<T, false>), dim3((unsigned)nblk), dim3(256), 0, st, in, out, rows, cols, drop);
  return hipGetLastError();
}

}  // namespace varuna
