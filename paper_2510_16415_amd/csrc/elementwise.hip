// HBM-bound kernels of the degraded block backward: RMSNorm recompute and backward with
// the residual add (the skip: dX = dOut + normbwd(dU)), the gain-gradient column
// reduction, the split-K reduction of the Eq. (2) token contraction, and the standalone
// SwiGLU backward used when saved activations are supplied.
// One wavefront (64 lanes) owns a row; row reductions are DPP/shuffle butterflies.
#include <type_traits>

#include "mecefo_internal.h"

namespace mecefo {
namespace {

template <typename T> __device__ inline float ldf(const T* p) { return (float)*p; }

__device__ inline float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Vector of VEC elements of T, loaded/stored with one instruction when VEC > 1.
template <typename T, int VEC> struct alignas(sizeof(T) * VEC) Vec { T e[VEC]; };

// One entry per thread, evaluated in fp64 and stored as fp32.
__device__ inline void rope_table_block(const RopeTables& t, unsigned block) {
  const int i = block * 256 + threadIdx.x;
  if (i >= t.seq * t.half) return;
  const int s = i / t.half, j = i - s * t.half;
  const double inv = pow(t.theta, -(double)j / (double)t.half);   // 2j / dh with dh = 2 * half
  const double ang = (double)s * inv;
  t.cs[i] = (float)cos(ang);
  t.sn[i] = (float)sin(ang);
}

// U = norm(H) gamma, a wave per row; the first `table_blocks` workgroups write the rotary tables instead.
template <typename T, int VEC>
__global__ __launch_bounds__(256) void rmsnorm_fwd_kernel(const T* __restrict__ H, int64_t ldh,
                                                          const T* __restrict__ gamma, float eps,
                                                          T* __restrict__ U, int64_t ldu,
                                                          float* __restrict__ rstd, int64_t b, int d,
                                                          RopeTables tables, unsigned table_blocks) {
  if (blockIdx.x < table_blocks) return rope_table_block(tables, blockIdx.x);
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)(blockIdx.x - table_blocks) * 4 + (threadIdx.x >> 6);
  if (row >= b) return;
  const T* h = H + row * ldh;
  const int nv = d / VEC;
  float ss = 0.f;
  for (int i = lane; i < nv; i += 64) {
    const Vec<T, VEC> x = *(const Vec<T, VEC>*)(h + i * VEC);
#pragma unroll
    for (int e = 0; e < VEC; ++e) { const float f = (float)x.e[e]; ss += f * f; }
  }
  ss = wave_sum(ss);
  const float rs = 1.0f / sqrtf(ss / (float)d + eps);
  if (lane == 0) rstd[row] = rs;
  T* u = U + row * ldu;
  for (int i = lane; i < nv; i += 64) {
    const Vec<T, VEC> x = *(const Vec<T, VEC>*)(h + i * VEC);
    const Vec<T, VEC> g = *(const Vec<T, VEC>*)(gamma + i * VEC);
    Vec<T, VEC> o;
#pragma unroll
    for (int e = 0; e < VEC; ++e) o.e[e] = (T)((float)x.e[e] * rs * (float)g.e[e]);
    *(Vec<T, VEC>*)(u + i * VEC) = o;
  }
}

// The same with the row held in registers between the two passes (ITERS vectors per lane cover the
// row): one read of H from memory, nothing re-read through the caches.
template <typename T, int VEC, int ITERS>
__global__ __launch_bounds__(256) void rmsnorm_fwd_row_kernel(const T* __restrict__ H, int64_t ldh,
                                                              const T* __restrict__ gamma, float eps,
                                                              T* __restrict__ U, int64_t ldu,
                                                              float* __restrict__ rstd, int64_t b, int d,
                                                              RopeTables tables, unsigned table_blocks) {
  if (blockIdx.x < table_blocks) return rope_table_block(tables, blockIdx.x);
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)(blockIdx.x - table_blocks) * 4 + (threadIdx.x >> 6);
  if (row >= b) return;
  const T* h = H + row * ldh;
  const int nv = d / VEC;
  Vec<T, VEC> x[ITERS];
  float ss = 0.f;
#pragma unroll
  for (int k = 0; k < ITERS; ++k) {
    const int i = k * 64 + lane;
    if (i < nv) {
      x[k] = *(const Vec<T, VEC>*)(h + i * VEC);
#pragma unroll
      for (int e = 0; e < VEC; ++e) { const float f = (float)x[k].e[e]; ss += f * f; }
    }
  }
  ss = wave_sum(ss);
  const float rs = 1.0f / sqrtf(ss / (float)d + eps);
  if (lane == 0) rstd[row] = rs;
  T* u = U + row * ldu;
#pragma unroll
  for (int k = 0; k < ITERS; ++k) {
    const int i = k * 64 + lane;
    if (i < nv) {
      const Vec<T, VEC> g = *(const Vec<T, VEC>*)(gamma + i * VEC);
      Vec<T, VEC> o;
#pragma unroll
      for (int e = 0; e < VEC; ++e) o.e[e] = (T)((float)x[k].e[e] * rs * (float)g.e[e]);
      *(Vec<T, VEC>*)(u + i * VEC) = o;
    }
  }
}

// dX_i = dOut_i + rstd_i * (dN_i - N_i * mean_j(dN_ij N_ij)),  dN = dU*gamma, N = H*rstd.
template <typename T, int VEC>
__global__ __launch_bounds__(256) void rmsnorm_bwd_kernel(const T* __restrict__ dU, int64_t lddu,
                                                          const T* __restrict__ H, int64_t ldh,
                                                          const float* __restrict__ rstd,
                                                          const T* __restrict__ gamma,
                                                          const T* dOut, int64_t lddo, T* dX, int64_t lddx,
                                                          int64_t b, int d) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= b) return;
  const T* du = dU + row * lddu;
  const T* h = H + row * ldh;
  const float rs = rstd[row];
  const int nv = d / VEC;
  float dot = 0.f;
  for (int i = lane; i < nv; i += 64) {
    const Vec<T, VEC> a = *(const Vec<T, VEC>*)(du + i * VEC);
    const Vec<T, VEC> x = *(const Vec<T, VEC>*)(h + i * VEC);
    const Vec<T, VEC> g = *(const Vec<T, VEC>*)(gamma + i * VEC);
#pragma unroll
    for (int e = 0; e < VEC; ++e) dot += (float)a.e[e] * (float)g.e[e] * ((float)x.e[e] * rs);
  }
  const float c = wave_sum(dot) / (float)d;
  const T* go = dOut + row * lddo;
  T* dx = dX + row * lddx;
  for (int i = lane; i < nv; i += 64) {
    const Vec<T, VEC> a = *(const Vec<T, VEC>*)(du + i * VEC);
    const Vec<T, VEC> x = *(const Vec<T, VEC>*)(h + i * VEC);
    const Vec<T, VEC> g = *(const Vec<T, VEC>*)(gamma + i * VEC);
    const Vec<T, VEC> r = *(const Vec<T, VEC>*)(go + i * VEC);
    Vec<T, VEC> o;
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      const float n = (float)x.e[e] * rs;
      o.e[e] = (T)((float)r.e[e] + rs * ((float)a.e[e] * (float)g.e[e] - n * c));
    }
    *(Vec<T, VEC>*)(dx + i * VEC) = o;
  }
}

// Rows per workgroup of the norm backward, and so rows per entry of its gain-gradient partials.
constexpr int kDgammaRows = 16;

// Norm backward, residual add and the gain-gradient partials in one pass over dU, H and dOut: a
// workgroup owns kDgammaRows consecutive rows, each of its four waves four of them.  2048 to 8192 rows are
// only 128 to 512 workgroups, so a wave's rows one after the other, a memory latency each, set the time
// (11 us for [4096 x 1024], 6.9 us for [2048 x 512]); here a wave has all four rows in flight at once
// (the 8-layer stack of the latter 1371 -> 1362 us, the two calls of the former 550 -> 549).  Rows of dU, H and dOut stay in registers (ITERS vectors per lane and row), and
// every lane sums dU * N of its columns over the wave's rows.  The four waves' sums are combined through LDS in
// a fixed order into partial[block][col] (results do not depend on scheduling).  partial may be NULL.
template <typename T, int VEC, int ITERS>
__global__ __launch_bounds__(256, 2) void rmsnorm_bwd_fused_kernel(const T* __restrict__ dU, int64_t lddu,
                                                                   const T* __restrict__ H, int64_t ldh,
                                                                   const float* __restrict__ rstd,
                                                                   const T* __restrict__ gamma,
                                                                   const T* dOut, int64_t lddo, T* dX, int64_t lddx,
                                                                   float* __restrict__ partial, int64_t b, int d) {
  extern __shared__ float comb[];      // [3][d]: the column sums of waves 1-3
  constexpr int RB = kDgammaRows / 4;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int nv = d / VEC;
  const int64_t r0 = (int64_t)blockIdx.x * kDgammaRows + wave;
  // rows r0, r0 + 4, ...: all are read before the first of them is written (dX may be dOut).  The loads carry no
  // branch (rows and columns outside the matrix read the last row or first column, unused): behind a branch
  // the compiler waits for each load before the next.
  Vec<T, VEC> g[ITERS], a[RB][ITERS], x[RB][ITERS], r[RB][ITERS];
  float rs[RB];
#pragma unroll
  for (int q = 0; q < RB; ++q) {
    const int64_t row = r0 + 4 * q < b ? r0 + 4 * q : b - 1;
    rs[q] = rstd[row];
#pragma unroll
    for (int k = 0; k < ITERS; ++k) {
      const int i = k * 64 + lane < nv ? k * 64 + lane : 0;
      a[q][k] = *(const Vec<T, VEC>*)(dU + row * lddu + i * VEC);
      x[q][k] = *(const Vec<T, VEC>*)(H + row * ldh + i * VEC);
      r[q][k] = *(const Vec<T, VEC>*)(dOut + row * lddo + i * VEC);
    }
  }
  float acc[ITERS][VEC];
#pragma unroll
  for (int k = 0; k < ITERS; ++k) {
    g[k] = *(const Vec<T, VEC>*)(gamma + (k * 64 + lane < nv ? k * 64 + lane : 0) * VEC);
#pragma unroll
    for (int e = 0; e < VEC; ++e) acc[k][e] = 0.f;
  }
#pragma unroll
  for (int q = 0; q < RB; ++q) {
    const int64_t row = r0 + 4 * q;
    if (row >= b) break;               // the same for the whole wave
    float dot = 0.f;
#pragma unroll
    for (int k = 0; k < ITERS; ++k) {
      float s = 0.f;
#pragma unroll
      for (int e = 0; e < VEC; ++e) s += (float)a[q][k].e[e] * (float)g[k].e[e] * ((float)x[q][k].e[e] * rs[q]);
      dot += k * 64 + lane < nv ? s : 0.f;
    }
    const float c = wave_sum(dot) / (float)d;
    T* dx = dX + row * lddx;
#pragma unroll
    for (int k = 0; k < ITERS; ++k) {
      const int i = k * 64 + lane;
      if (i < nv) {
        Vec<T, VEC> o;
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
          const float n = (float)x[q][k].e[e] * rs[q];
          o.e[e] = (T)((float)r[q][k].e[e] + rs[q] * ((float)a[q][k].e[e] * (float)g[k].e[e] - n * c));
          acc[k][e] += (float)a[q][k].e[e] * n;
        }
        *(Vec<T, VEC>*)(dx + i * VEC) = o;
      }
    }
  }
  if (!partial) return;      // kernel argument: the whole workgroup takes the same branch
  if (wave > 0) {
#pragma unroll
    for (int k = 0; k < ITERS; ++k) {
      const int i = k * 64 + lane;
      if (i < nv) {
#pragma unroll
        for (int e = 0; e < VEC; ++e) comb[(wave - 1) * d + i * VEC + e] = acc[k][e];
      }
    }
  }
  __syncthreads();
  if (wave == 0) {
#pragma unroll
    for (int k = 0; k < ITERS; ++k) {
      const int i = k * 64 + lane;
      if (i < nv) {
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
          const int col = i * VEC + e;
          partial[(int64_t)blockIdx.x * d + col] = ((acc[k][e] + comb[col]) + comb[d + col]) + comb[2 * d + col];
        }
      }
    }
  }
}

// The same for long rows: the whole workgroup works on RB rows at a time (thread t owns vectors
// t, t + 256, ...), the row dot products are combined across the four waves through LDS (one barrier
// per group of rows, alternating slots), and the next group's rows are fetched while the current one is
// finished.  RB keeps about four vectors of each operand per thread in flight and a barrier per RB rows, 8 to 16 KB
// of each operand (one row at a time: 21 us for [2048 x 2048]; the skip call around it went from 465 to 458 us, the standard
// one with two of them from 757 to 739).  Every thread owns its columns for all rows
// of the block, so its sums go straight to partial[block][col].
template <typename T, int VEC, int ITERS, int RB>
__global__ __launch_bounds__(256) void rmsnorm_bwd_block_kernel(const T* __restrict__ dU, int64_t lddu,
                                                                const T* __restrict__ H, int64_t ldh,
                                                                const float* __restrict__ rstd,
                                                                const T* __restrict__ gamma,
                                                                const T* dOut, int64_t lddo, T* dX, int64_t lddx,
                                                                float* __restrict__ partial, int64_t b, int d) {
  __shared__ float red[2][RB][4];
  static_assert(kDgammaRows % (2 * RB) == 0, "two groups per turn of the loop");
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int nv = d / VEC;
  struct Rows { Vec<T, VEC> a[RB][ITERS], x[RB][ITERS], r[RB][ITERS]; float rs[RB]; };
  Vec<T, VEC> g[ITERS];
  float acc[ITERS][VEC];
#pragma unroll
  for (int k = 0; k < ITERS; ++k) {
    g[k] = *(const Vec<T, VEC>*)(gamma + (k * 256 + t < nv ? k * 256 + t : 0) * VEC);
#pragma unroll
    for (int e = 0; e < VEC; ++e) acc[k][e] = 0.f;
  }
  const int64_t r0 = (int64_t)blockIdx.x * kDgammaRows;
  const int64_t r1 = r0 + kDgammaRows < b ? r0 + kDgammaRows : b;
  // dOut of a row is read before the store of that row's dX, which may be the same memory; a group's stores
  // never precede the reads of its own rows.  No branch around the loads (see above).
  auto fetch = [&](int64_t row0, Rows& w) {
#pragma unroll
    for (int q = 0; q < RB; ++q) {
      const int64_t row = row0 + q < r1 ? row0 + q : r1 - 1;
      w.rs[q] = rstd[row];
#pragma unroll
      for (int k = 0; k < ITERS; ++k) {
        const int i = k * 256 + t < nv ? k * 256 + t : 0;
        w.a[q][k] = *(const Vec<T, VEC>*)(dU + row * lddu + i * VEC);
        w.x[q][k] = *(const Vec<T, VEC>*)(H + row * ldh + i * VEC);
        w.r[q][k] = *(const Vec<T, VEC>*)(dOut + row * lddo + i * VEC);
      }
    }
  };
  auto finish = [&](int64_t row0, int slot, const Rows& w) {
#pragma unroll
    for (int q = 0; q < RB; ++q) {
      float dot = 0.f;
#pragma unroll
      for (int k = 0; k < ITERS; ++k) {
        float s = 0.f;
#pragma unroll
        for (int e = 0; e < VEC; ++e) s += (float)w.a[q][k].e[e] * (float)g[k].e[e] * ((float)w.x[q][k].e[e] * w.rs[q]);
        dot += k * 256 + t < nv ? s : 0.f;
      }
      dot = wave_sum(dot);
      if (lane == 0) red[slot][q][wave] = dot;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < RB; ++q) {
      if (row0 + q >= r1) break;
      const float c = ((red[slot][q][0] + red[slot][q][1]) + (red[slot][q][2] + red[slot][q][3])) / (float)d;
      T* dx = dX + (row0 + q) * lddx;
#pragma unroll
      for (int k = 0; k < ITERS; ++k) {
        const int i = k * 256 + t;
        if (i < nv) {
          Vec<T, VEC> o;
#pragma unroll
          for (int e = 0; e < VEC; ++e) {
            const float n = (float)w.x[q][k].e[e] * w.rs[q];
            o.e[e] = (T)((float)w.r[q][k].e[e] + w.rs[q] * ((float)w.a[q][k].e[e] * (float)g[k].e[e] - n * c));
            acc[k][e] += (float)w.a[q][k].e[e] * n;
          }
          *(Vec<T, VEC>*)(dx + i * VEC) = o;
        }
      }
    }
  };
  // Two register sets take turns (no copies between them: a copy would have to wait for the loads
  // it moves): one group is finished from the first while the second receives the group after it.
  Rows w0, w1;
  fetch(r0, w0);
#pragma unroll 1
  for (int64_t row = r0; row < r1; row += 2 * RB) {      // bounds are the same for the whole workgroup
    fetch(row + RB, w1);
    finish(row, 0, w0);
    fetch(row + 2 * RB, w0);
    if (row + RB < r1) finish(row + RB, 1, w1);
  }
  if (!partial) return;
#pragma unroll
  for (int k = 0; k < ITERS; ++k) {
    const int i = k * 256 + t;
    if (i < nv) {
#pragma unroll
      for (int e = 0; e < VEC; ++e) partial[(int64_t)blockIdx.x * d + i * VEC + e] = acc[k][e];
    }
  }
}

// The same with a wave per row and as few rows per workgroup as it takes to fill the chip (rpw rows per wave, one after
// the other); dU comes in the storage type (NP = 0), or as the NP fp32 parts of a product that was cut along K, added up
// here in their order: a launch that sums them, and a bf16 rounding, are saved.  [2048 x 2048] from three parts: 11.5 us for the
// sum and 14.5 behind it before, 17.7 now (76 MB); fp32 [256 x 256]: two launches of 9 us in all before, 5.0 now.
template <typename T, int VEC, int ITERS, int NP>
__global__ __launch_bounds__(256) void rmsnorm_bwd_rows_kernel(const void* __restrict__ dU, int64_t lddu, int64_t part,
                                                               const T* __restrict__ H, int64_t ldh,
                                                               const float* __restrict__ rstd,
                                                               const T* __restrict__ gamma,
                                                               const T* dOut, int64_t lddo, T* dX, int64_t lddx,
                                                               float* __restrict__ partial, int64_t b, int d, int rpw) {
  extern __shared__ float comb[];      // [3][d]: the column sums of waves 1-3
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int nv = d / VEC;
  Vec<T, VEC> g[ITERS];
  float acc[ITERS][VEC];
#pragma unroll
  for (int k = 0; k < ITERS; ++k) {
    g[k] = *(const Vec<T, VEC>*)(gamma + (k * 64 + lane < nv ? k * 64 + lane : 0) * VEC);
#pragma unroll
    for (int e = 0; e < VEC; ++e) acc[k][e] = 0.f;
  }
#pragma unroll 1
  for (int q = 0; q < rpw; ++q) {
    const int64_t row = (int64_t)blockIdx.x * 4 * rpw + 4 * q + wave;
    if (row >= b) break;               // the same for the whole wave
    // no branch around the loads (see above); all of a row are read before it is written (dX may be dOut)
    float a[ITERS][VEC];
    Vec<T, VEC> x[ITERS], r[ITERS];
#pragma unroll
    for (int k = 0; k < ITERS; ++k) {
      const int i = k * 64 + lane < nv ? k * 64 + lane : 0;
      x[k] = *(const Vec<T, VEC>*)(H + row * ldh + i * VEC);
      r[k] = *(const Vec<T, VEC>*)(dOut + row * lddo + i * VEC);
      if constexpr (NP == 0) {
        const Vec<T, VEC> v = *(const Vec<T, VEC>*)((const T*)dU + row * lddu + i * VEC);
#pragma unroll
        for (int e = 0; e < VEC; ++e) a[k][e] = (float)v.e[e];
      } else {
        constexpr int V4 = VEC < 4 ? VEC : 4;
        Vec<float, V4> v[NP][VEC / V4];
#pragma unroll
        for (int n = 0; n < NP; ++n)
#pragma unroll
          for (int h = 0; h < VEC / V4; ++h)
            v[n][h] = *(const Vec<float, V4>*)((const float*)dU + n * part + row * lddu + i * VEC + h * V4);
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
          a[k][e] = v[0][e / V4].e[e % V4];
#pragma unroll
          for (int n = 1; n < NP; ++n) a[k][e] += v[n][e / V4].e[e % V4];
        }
      }
    }
    const float rs = rstd[row];
    float dot = 0.f;
#pragma unroll
    for (int k = 0; k < ITERS; ++k) {
      float s = 0.f;
#pragma unroll
      for (int e = 0; e < VEC; ++e) s += a[k][e] * (float)g[k].e[e] * ((float)x[k].e[e] * rs);
      dot += k * 64 + lane < nv ? s : 0.f;
    }
    const float c = wave_sum(dot) / (float)d;
    T* dx = dX + row * lddx;
#pragma unroll
    for (int k = 0; k < ITERS; ++k) {
      const int i = k * 64 + lane;
      if (i < nv) {
        Vec<T, VEC> o;
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
          const float n = (float)x[k].e[e] * rs;
          o.e[e] = (T)((float)r[k].e[e] + rs * (a[k][e] * (float)g[k].e[e] - n * c));
          acc[k][e] += a[k][e] * n;
        }
        *(Vec<T, VEC>*)(dx + i * VEC) = o;
      }
    }
  }
  if (!partial) return;      // kernel argument: the whole workgroup takes the same branch
  if (wave > 0) {
#pragma unroll
    for (int k = 0; k < ITERS; ++k) {
      const int i = k * 64 + lane;
      if (i < nv) {
#pragma unroll
        for (int e = 0; e < VEC; ++e) comb[(wave - 1) * d + i * VEC + e] = acc[k][e];
      }
    }
  }
  __syncthreads();
  if (wave == 0) {
#pragma unroll
    for (int k = 0; k < ITERS; ++k) {
      const int i = k * 64 + lane;
      if (i < nv) {
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
          const int col = i * VEC + e;
          partial[(int64_t)blockIdx.x * d + col] = ((acc[k][e] + comb[col]) + comb[d + col]) + comb[2 * d + col];
        }
      }
    }
  }
}

// Partial column sums of dU * N over a chunk of rows: partial[chunk][col].
template <typename T, int VEC>
__global__ __launch_bounds__(256) void dgamma_partial_kernel(const T* __restrict__ dU, int64_t lddu,
                                                             const T* __restrict__ H, int64_t ldh,
                                                             const float* __restrict__ rstd,
                                                             float* __restrict__ partial, int64_t b, int d,
                                                             int rows_per_chunk) {
  const int cv = blockIdx.x * 256 + threadIdx.x;
  if (cv * VEC >= d) return;
  const int64_t r0 = (int64_t)blockIdx.y * rows_per_chunk;
  const int64_t r1 = r0 + rows_per_chunk < b ? r0 + rows_per_chunk : b;
  float acc[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) acc[e] = 0.f;
  for (int64_t r = r0; r < r1; ++r) {
    const Vec<T, VEC> a = *(const Vec<T, VEC>*)(dU + r * lddu + cv * VEC);
    const Vec<T, VEC> x = *(const Vec<T, VEC>*)(H + r * ldh + cv * VEC);
    const float rs = rstd[r];
#pragma unroll
    for (int e = 0; e < VEC; ++e) acc[e] += (float)a.e[e] * ((float)x.e[e] * rs);
  }
#pragma unroll
  for (int e = 0; e < VEC; ++e) partial[(int64_t)blockIdx.y * d + cv * VEC + e] = acc[e];
}

// dgamma[c] = sum over chunks of partial[chunk][c].  A block owns 32 columns; its 32 groups of 32
// threads each sum a strided part of the chunks (coalesced 128-byte rows), then combine in LDS
// in a fixed order.
template <typename T>
__global__ __launch_bounds__(1024) void dgamma_reduce_kernel(const float* __restrict__ partial, int nblk, int d,
                                                             void* dgamma, int out_f32, int accumulate) {
  __shared__ float red[32][32];
  const int cl = threadIdx.x & 31, g = threadIdx.x >> 5;
  const int c = blockIdx.x * 32 + cl;
  float s = 0.f;
  if (c < d) {
#pragma unroll 16
    for (int k = g; k < nblk; k += 32) s += partial[(int64_t)k * d + c];
  }
  red[g][cl] = s;
  __syncthreads();
  if (g != 0 || c >= d) return;
#pragma unroll
  for (int k = 1; k < 32; ++k) s += red[k][cl];
  if (out_f32) {
    float* o = (float*)dgamma;
    o[c] = accumulate ? o[c] + s : s;
  } else {
    T* o = (T*)dgamma;
    o[c] = (T)(accumulate ? (float)o[c] + s : s);
  }
}

template <typename T, int VEC>
__global__ __launch_bounds__(256) void add_kernel(const T* a, int64_t lda, const T* __restrict__ bsrc,
                                                  int64_t ldb, T* out, int64_t ldo, int64_t rows, int cols) {
  const int nv = cols / VEC;
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= rows * nv) return;
  const int64_t r = idx / nv;
  const int cv = (int)(idx - r * nv);
  const Vec<T, VEC> x = *(const Vec<T, VEC>*)(a + r * lda + cv * VEC);
  const Vec<T, VEC> y = *(const Vec<T, VEC>*)(bsrc + r * ldb + cv * VEC);
  Vec<T, VEC> o;
#pragma unroll
  for (int e = 0; e < VEC; ++e) o.e[e] = (T)((float)x.e[e] + (float)y.e[e]);
  *(Vec<T, VEC>*)(out + r * ldo + cv * VEC) = o;
}

// out[i] = sum over the parts of part[k][i] for up to four products, fixed summation order (bit-reproducible).  One
// launch for all of them: a launch of its own for each of three small products is 5 us each.
struct SumJobs { SumJob j[kMaxProblems]; unsigned first[kMaxProblems]; };      // first[k]: first block of job k
template <typename T>
__global__ __launch_bounds__(256) void sum_parts_kernel(const SumJobs a) {
  int k = 0;
#pragma unroll
  for (int i = 1; i < kMaxProblems; ++i) k = blockIdx.x >= a.first[i] ? i : k;
  const SumJob job = a.j[k];
  T* C = (T*)job.out;
  const int64_t i4 = ((int64_t)(blockIdx.x - a.first[k]) * 256 + threadIdx.x) * 4, mn = job.n;
  if (i4 >= mn) return;
  if (i4 + 4 <= mn && mn % 4 == 0) {
    float4 s = *(const float4*)(job.part + i4);
#pragma unroll 4
    for (int q = 1; q < job.parts; ++q) {
      const float4 v = *(const float4*)(job.part + (int64_t)q * mn + i4);
      s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
    }
    Vec<T, 4> o;
    o.e[0] = (T)s.x; o.e[1] = (T)s.y; o.e[2] = (T)s.z; o.e[3] = (T)s.w;
    *(Vec<T, 4>*)(C + i4) = o;
  } else {
    for (int64_t i = i4; i < mn && i < i4 + 4; ++i) {
      float s = 0.f;
      for (int q = 0; q < job.parts; ++q) s += job.part[(int64_t)q * mn + i];
      C[i] = (T)s;
    }
  }
}

template <bool PRECISE> __device__ inline float sigm(float g) {
  if constexpr (PRECISE) return 1.0f / (1.0f + expf(-g));
  else return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.44269504088896341f * g));
}

// dA (in DG), saved G, Z  ->  DG = dG, DZ = dZ, AA = silu(G)*Z.  VEC columns per thread.
template <typename T, int VEC>
__global__ __launch_bounds__(256) void swiglu_bwd_kernel(const T* __restrict__ G, const T* __restrict__ Z,
                                                         int64_t ldgz, T* DG, T* __restrict__ DZ,
                                                         T* __restrict__ AA, int64_t ldf, int64_t b, int f,
                                                         int pad_cols) {
  const int nv = (pad_cols + VEC - 1) / VEC;
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= b * nv) return;
  const int64_t r = idx / nv;
  const int c0 = (int)(idx - r * nv) * VEC;
  Vec<T, VEC> g, z, da, odg, odz, oa;
  if (c0 < f) {
    g = *(const Vec<T, VEC>*)(G + r * ldgz + c0);
    z = *(const Vec<T, VEC>*)(Z + r * ldgz + c0);
    da = *(const Vec<T, VEC>*)(DG + r * ldf + c0);
  }
#pragma unroll
  for (int e = 0; e < VEC; ++e) {
    float vdg = 0.f, vdz = 0.f, va = 0.f;
    if (c0 + e < f) {
      const float gg = (float)g.e[e], zz = (float)z.e[e], d = (float)da.e[e];
      const float sg = sigm<sizeof(T) == 4>(gg);
      const float s = gg * sg;
      va = s * zz;
      vdz = d * s;
      vdg = d * zz * (sg * (1.0f + gg * (1.0f - sg)));
    }
    odg.e[e] = (T)vdg; odz.e[e] = (T)vdz; oa.e[e] = (T)va;
  }
  *(Vec<T, VEC>*)(DG + r * ldf + c0) = odg;
  *(Vec<T, VEC>*)(DZ + r * ldf + c0) = odz;
  *(Vec<T, VEC>*)(AA + r * ldf + c0) = oa;
}

inline unsigned blocks_for(int64_t n) { return (unsigned)((n + 255) / 256); }

// The register-resident row kernels (bf16, eight elements per lane and step) cover rows of up to
// 8 * 64 * 8 = 4096 elements whose strides keep every 16-byte vector aligned.
bool row_fits(int d, int64_t l0, int64_t l1, int64_t l2, int64_t l3) {
  return d % 8 == 0 && d <= 4096 && l0 % 8 == 0 && l1 % 8 == 0 && l2 % 8 == 0 && l3 % 8 == 0;
}
template <typename F> void dispatch_iters(int nv, F&& f) {
  if (nv <= 64) f(std::integral_constant<int, 1>{});
  else if (nv <= 128) f(std::integral_constant<int, 2>{});
  else if (nv <= 256) f(std::integral_constant<int, 4>{});
  else f(std::integral_constant<int, 8>{});
}

}  // namespace

hipError_t launch_rmsnorm_fwd(bool bf16, const void* H, int64_t ldh, const void* gamma, float eps, void* U,
                              int64_t ldu, float* rstd, int64_t b, int d, hipStream_t s,
                              const RopeTables* tables) {
  const RopeTables t = tables ? *tables : RopeTables{};
  const unsigned nt = rope_table_blocks(t), grid = nt + (unsigned)((b + 3) / 4);
  if (bf16 && row_fits(d, ldh, ldu, ldu, ldu)) {
    auto go = [&](auto iters) {
      hipLaunchKernelGGL((rmsnorm_fwd_row_kernel<__bf16, 8, decltype(iters)::value>), dim3(grid), dim3(256), 0, s,
                         (const __bf16*)H, ldh, (const __bf16*)gamma, eps, (__bf16*)U, ldu, rstd, b, d, t, nt);
    };
    dispatch_iters(d / 8, go);
  } else if (bf16)
    hipLaunchKernelGGL((rmsnorm_fwd_kernel<__bf16, 8>), dim3(grid), dim3(256), 0, s, (const __bf16*)H, ldh,
                       (const __bf16*)gamma, eps, (__bf16*)U, ldu, rstd, b, d, t, nt);
  else
    hipLaunchKernelGGL((rmsnorm_fwd_kernel<float, 1>), dim3(grid), dim3(256), 0, s, (const float*)H, ldh,
                       (const float*)gamma, eps, (float*)U, ldu, rstd, b, d, t, nt);
  return hipGetLastError();
}

int rmsnorm_bwd_blocks(int64_t b) { return (int)((b + kDgammaRows - 1) / kDgammaRows); }

namespace {
// What the kernel with a wave per row reads: vectors of 16 bytes where everything is aligned to them, single fp32
// elements of short rows where not; 0 where it is not built.
int rows_kernel_vec(bool bf16, const NormBwd& n) {
  const int v = bf16 ? 8 : 4;
  const uintptr_t bits = (uintptr_t)n.dU | (uintptr_t)n.H | (uintptr_t)n.gamma | (uintptr_t)n.dOut | (uintptr_t)n.dX;
  const bool aligned = n.lddu % v == 0 && n.ldh % v == 0 && n.lddo % v == 0 && n.lddx % v == 0 && bits % 16 == 0;
  if (aligned && rmsnorm_bwd_parts_width(bf16, n.d)) return v;
  return !bf16 && n.parts == 0 && n.d <= 512 ? 1 : 0;
}
// Rows per wave: few enough for 512 workgroups, as far as there is room for a row of gain-gradient sums from each.
int rows_kernel_rpw(const NormBwd& n) {
  int rpw = 1;
  while (rpw < 4 && (n.b + 4 * rpw - 1) / (4 * rpw) > 512) rpw *= 2;
  while (rpw < 4 && n.dg_partial && (n.b + 4 * rpw - 1) / (4 * rpw) * n.d > n.dg_room) rpw *= 2;
  return rpw;
}
}  // namespace

bool rmsnorm_bwd_takes_parts(bool bf16, const NormBwd& n) {
  return n.parts >= 2 && n.parts <= kMaxNormParts && rows_kernel_vec(bf16, n) > 1;
}

hipError_t launch_rmsnorm_bwd(bool bf16, const NormBwd& n, int* nblk, hipStream_t s) {
  const int64_t b = n.b;
  const int d = n.d;
  const int vec = rows_kernel_vec(bf16, n);
  // bf16 without parts: more rows per wave go to the kernels that have several of them in flight
  const int rpw = rows_kernel_rpw(n);
  if (vec > 0 && (n.parts > 0 || !bf16 || rpw <= 2)) {
    *nblk = (int)((b + 4 * rpw - 1) / (4 * rpw));
    auto go = [&](auto type, auto v, auto iters, auto np) {
      using T = decltype(type);
      hipLaunchKernelGGL((rmsnorm_bwd_rows_kernel<T, decltype(v)::value, decltype(iters)::value, decltype(np)::value>),
                         dim3((unsigned)*nblk), dim3(256), (size_t)3 * d * 4, s, n.dU, n.lddu, n.part_stride, (const T*)n.H, n.ldh,
                         n.rstd, (const T*)n.gamma, (const T*)n.dOut, n.lddo, (T*)n.dX, n.lddx, n.dg_partial, b, d, rpw);
    };
    auto parts = [&](auto type, auto v, auto iters) {
      if (n.parts == 2) go(type, v, iters, std::integral_constant<int, 2>{});
      else if (n.parts == 3) go(type, v, iters, std::integral_constant<int, 3>{});
      else if (n.parts == 4) go(type, v, iters, std::integral_constant<int, 4>{});
      else go(type, v, iters, std::integral_constant<int, 0>{});
    };
    if (bf16) dispatch_iters(d / 8, [&](auto iters) {
      if constexpr (decltype(iters)::value <= 4) parts(__bf16{}, std::integral_constant<int, 8>{}, iters);
    });
    else if (vec == 4) dispatch_iters(d / 4, [&](auto iters) { parts(float{}, std::integral_constant<int, 4>{}, iters); });
    else go(float{}, std::integral_constant<int, 1>{}, std::integral_constant<int, 8>{}, std::integral_constant<int, 0>{});
    return hipGetLastError();
  }
  *nblk = rmsnorm_bwd_blocks(b);
  if (n.parts > 0) return hipErrorInvalidValue;
  if (bf16 && d % 8 == 0 && d <= 8192 && n.lddu % 8 == 0 && n.ldh % 8 == 0 && n.lddo % 8 == 0 && n.lddx % 8 == 0) {
    const int nv = d / 8;
    const dim3 grid((unsigned)*nblk);
#define MECEFO_NORM_BWD(LDS, ...)                                                                                    \
  hipLaunchKernelGGL((__VA_ARGS__), grid, dim3(256), LDS, s, (const __bf16*)n.dU, n.lddu, (const __bf16*)n.H, n.ldh, n.rstd,   \
                     (const __bf16*)n.gamma, (const __bf16*)n.dOut, n.lddo, (__bf16*)n.dX, n.lddx, n.dg_partial, b, d)
    const size_t comb = (size_t)3 * d * 4;
    if (nv <= 64) MECEFO_NORM_BWD(comb, rmsnorm_bwd_fused_kernel<__bf16, 8, 1>);         // a wave per row
    else if (nv <= 128) MECEFO_NORM_BWD(comb, rmsnorm_bwd_fused_kernel<__bf16, 8, 2>);
    else if (nv <= 256) MECEFO_NORM_BWD(0, rmsnorm_bwd_block_kernel<__bf16, 8, 1, 4>);   // the workgroup per row
    else if (nv <= 512) MECEFO_NORM_BWD(0, rmsnorm_bwd_block_kernel<__bf16, 8, 2, 2>);
    else MECEFO_NORM_BWD(0, rmsnorm_bwd_block_kernel<__bf16, 8, 4, 1>);
#undef MECEFO_NORM_BWD
    return hipGetLastError();
  }
  // The gain-gradient partials read dU and H before dX is written (dX may alias dOut only).
  if (n.dg_partial) {
    if (bf16)
      hipLaunchKernelGGL((dgamma_partial_kernel<__bf16, 8>), dim3(blocks_for(d / 8), *nblk), dim3(256), 0, s,
                         (const __bf16*)n.dU, n.lddu, (const __bf16*)n.H, n.ldh, n.rstd, n.dg_partial, b, d, kDgammaRows);
    else
      hipLaunchKernelGGL((dgamma_partial_kernel<float, 1>), dim3(blocks_for(d), *nblk), dim3(256), 0, s,
                         (const float*)n.dU, n.lddu, (const float*)n.H, n.ldh, n.rstd, n.dg_partial, b, d, kDgammaRows);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  const unsigned grid = (unsigned)((b + 3) / 4);
  if (bf16)
    hipLaunchKernelGGL((rmsnorm_bwd_kernel<__bf16, 8>), dim3(grid), dim3(256), 0, s, (const __bf16*)n.dU, n.lddu,
                       (const __bf16*)n.H, n.ldh, n.rstd, (const __bf16*)n.gamma, (const __bf16*)n.dOut, n.lddo,
                       (__bf16*)n.dX, n.lddx, b, d);
  else
    hipLaunchKernelGGL((rmsnorm_bwd_kernel<float, 1>), dim3(grid), dim3(256), 0, s, (const float*)n.dU, n.lddu,
                       (const float*)n.H, n.ldh, n.rstd, (const float*)n.gamma, (const float*)n.dOut, n.lddo, (float*)n.dX,
                       n.lddx, b, d);
  return hipGetLastError();
}

hipError_t launch_dgamma_reduce(const float* dg_partial, int nblk, int d, void* dgamma, bool out_f32,
                                bool bf16, int accumulate, hipStream_t s) {
  if (bf16)
    hipLaunchKernelGGL(dgamma_reduce_kernel<__bf16>, dim3((d + 31) / 32), dim3(1024), 0, s, dg_partial, nblk, d,
                       dgamma, (int)out_f32, accumulate);
  else
    hipLaunchKernelGGL(dgamma_reduce_kernel<float>, dim3((d + 31) / 32), dim3(1024), 0, s, dg_partial, nblk, d,
                       dgamma, 1, accumulate);
  return hipGetLastError();
}

hipError_t launch_add(bool bf16, const void* a, int64_t lda, const void* bsrc, int64_t ldb, void* out,
                      int64_t ldo, int64_t rows, int cols, hipStream_t s) {
  if (bf16)
    hipLaunchKernelGGL((add_kernel<__bf16, 8>), dim3(blocks_for(rows * (cols / 8))), dim3(256), 0, s,
                       (const __bf16*)a, lda, (const __bf16*)bsrc, ldb, (__bf16*)out, ldo, rows, cols);
  else
    hipLaunchKernelGGL((add_kernel<float, 1>), dim3(blocks_for(rows * cols)), dim3(256), 0, s, (const float*)a,
                       lda, (const float*)bsrc, ldb, (float*)out, ldo, rows, cols);
  return hipGetLastError();
}

hipError_t launch_sum_parts(bool bf16, const SumJob* jobs, int n, hipStream_t s) {
  SumJobs a;
  unsigned grid = 0;
  for (int i = 0; i < kMaxProblems; ++i) {
    a.j[i] = jobs[i < n ? i : 0];
    a.first[i] = i < n ? grid : 0xFFFFFFFFu;
    if (i < n) grid += blocks_for((jobs[i].n + 3) / 4);
  }
  if (grid == 0) return hipSuccess;
  if (bf16) hipLaunchKernelGGL(sum_parts_kernel<__bf16>, dim3(grid), dim3(256), 0, s, a);
  else hipLaunchKernelGGL(sum_parts_kernel<float>, dim3(grid), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_swiglu_bwd(bool bf16, const void* G, const void* Z, int64_t ldgz, void* DG, void* DZ,
                             void* AA, int64_t ldf, int64_t b, int f, int pad_cols, hipStream_t s) {
  if (bf16) {
    const int nv = (pad_cols + 7) / 8;
    hipLaunchKernelGGL((swiglu_bwd_kernel<__bf16, 8>), dim3(blocks_for(b * nv)), dim3(256), 0, s,
                       (const __bf16*)G, (const __bf16*)Z, ldgz, (__bf16*)DG, (__bf16*)DZ, (__bf16*)AA, ldf, b,
                       f, pad_cols);
  } else {
    hipLaunchKernelGGL((swiglu_bwd_kernel<float, 1>), dim3(blocks_for(b * pad_cols)), dim3(256), 0, s,
                       (const float*)G, (const float*)Z, ldgz, (float*)DG, (float*)DZ, (float*)AA, ldf, b, f,
                       pad_cols);
  }
  return hipGetLastError();
}

}  // namespace mecefo
