// Device-side pieces shared by the bf16 MFMA GEMM and the fp32 GEMM: kernel argument
// block, block-id -> tile mapping, and the per-element epilogues.
#pragma once
#include <stddef.h>

#include "mecefo_internal.h"

namespace mecefo {

// One problem as the kernels read it: two lines of 64 bytes.
struct KProblem {
  const void* A[3];
  const void* B[3];
  void* C[3];
  int64_t lda, ldb, ldc;
  int M, N, K;
  int chunk_nseg;          // 4 * (K stages of a workgroup) + nseg
  int aux;                 // EPI_ROPE: rope_half, else pad_cols
  int splits_kpad;         // 2 * splits + kpad_ok
  uint32_t by_tiles, by_group;   // div_magic of the tiles of one part or product, and of the tiles of eight tile rows
};

// Division by a number that the host knows: one multiplication and a correction, where the compiler's sequence is
// 30 instructions.
inline uint32_t div_magic(uint32_t n) { return n > 1 ? (uint32_t)(((uint64_t)1 << 32) / n + 1) : 0xFFFFFFFFu; }
__host__ __device__ inline int div_by(int x, int n, uint32_t magic) {
  // n > 1: magic - 2^32 / n lies in (0, 1], so the product is x / n plus less than 1; n = 1: x - 1 (0 for x = 0)
  const int q = (int)(((uint64_t)(uint32_t)x * magic) >> 32), r = x - q * n;
  return q + (r >= n ? 1 : 0) - (r < 0 ? 1 : 0);
}

// Kernel arguments.  A workgroup needs them before its first load, and what it does until then is much of a small
// launch: a head that is fetched as a whole, the mapping to a tile from it, and the tile's problem, fetched as a whole.
// Fetched field by field, each where it is used, with the compiler's divisions in the mapping, the 64 x 64 store kernel had
// 673 instructions and 8 waits in front of its first fill; now it has 460 and 3.
struct KHead {
  int nprob, total;        // problems; workgroups: the sum over problems of tiles * splits (* batch)
  int accumulate, out_f32;
  int gemm_blocks;         // workgroups of the products; those behind them run the side job
  int order;               // problem indices, four bits each, most work per workgroup first
  int units[kMaxProblems]; // workgroups of the problems in that order
  int batch, batch_inner, causal, rope_seq;
  float scale, poly_a, poly_b;
  int tail;                // launches that cut up their last round: problem, log2 of the parts of a tile, first tile;
                           // EPI_HILO: fold_norm
  uint32_t* clk;           // measurement (NULL otherwise): every 64th workgroup stores its shader-clock cycles and
                           // its 100 MHz wall ticks, pair number (workgroup / 64) % 64
  const float* rowvec;
  const float* addend;
  int64_t a_bi, b_bi, c_bi, a_bo;
};
struct KArgs {
  KHead h;
  KProblem p[kMaxProblems];
  int64_t b_bo, c_bo;
  SideJob side;
};
static_assert(sizeof(KHead) == 128 && sizeof(KProblem) == 128 && offsetof(KArgs, p) == 128, "whole lines of 64 bytes");

// Host side: the arguments of a launch whose workgroups compute bm x bn tiles of the outputs in K stages of bk.  The logical
// order of the workgroups is eight consecutive segments, one per XCD; segment x lists, heaviest problem first, the
// x-th eighth of every problem's workgroups.  Longest-processing-time-first inside each segment keeps the tail of a
// grouped launch short when the problems differ in K.
inline void fill_kargs(KArgs& args, const GemmLaunch& g, int bm, int bn, int bk) {
  KHead& a = args.h;
  a.nprob = g.nprob;
  a.accumulate = g.accumulate;
  a.out_f32 = g.out_f32;
  a.clk = g.clk;
  const GemmProblem& f = g.p[0];      // what every problem of a launch shares
  a.batch = f.batch; a.batch_inner = f.batch_inner; a.causal = f.causal; a.rope_seq = f.rope_seq;
  a.scale = f.scale; a.poly_a = f.poly_a; a.poly_b = f.poly_b;
  a.tail = f.fold_norm;
  a.rowvec = f.rowvec; a.addend = f.addend;
  a.a_bo = f.a_bo; a.a_bi = f.a_bi; a.b_bi = f.b_bi; a.c_bi = f.c_bi;
  args.b_bo = f.b_bo; args.c_bo = f.c_bo;
  int idx[kMaxProblems], units[kMaxProblems];
  double work[kMaxProblems];
  a.total = 0;
  for (int i = 0; i < kMaxProblems; ++i) {
    const GemmProblem& p = g.p[i < g.nprob ? i : 0];
    KProblem& k = args.p[i];
    // dual products keep B[1] as the up matrix; unused segments repeat the first
    const bool dual = g.epi == EPI_SWIGLU_FWD || g.epi == EPI_SWIGLU_BWD;
    const int nseg = dual || p.nseg < 1 ? 1 : p.nseg, splits = p.splits > 1 ? p.splits : 1;
    for (int s = 0; s < 3; ++s) {
      k.A[s] = p.A[s < nseg ? s : 0];
      k.B[s] = p.B[s < (dual ? 2 : nseg) ? s : 0];
      k.C[s] = p.C[s];
    }
    k.lda = p.lda; k.ldb = p.ldb; k.ldc = p.ldc;
    k.M = p.M; k.N = p.N; k.K = p.K;
    const int stages = (p.K + bk - 1) / bk * nseg;
    k.chunk_nseg = 4 * ((stages + splits - 1) / splits) + nseg;
    k.aux = g.epi == EPI_ROPE ? p.rope_half : p.pad_cols;
    k.splits_kpad = 2 * splits + (p.kpad_ok ? 1 : 0);
    const int tiles_m = (p.M + bm - 1) / bm, tiles_n = (p.N + bn - 1) / bn;
    k.by_tiles = div_magic(tiles_m * tiles_n);
    k.by_group = div_magic(8 * tiles_n);
    idx[i] = i;
    units[i] = i < g.nprob ? tiles_m * tiles_n * splits * (p.batch > 1 ? p.batch : 1) : 0;
    work[i] = i < g.nprob ? (double)p.K * nseg / splits : -1.0;
    a.total += units[i];
  }
  for (int i = 0; i < kMaxProblems; ++i)      // stable: equal problems keep their order
    for (int j = kMaxProblems - 1; j > i; --j)
      if (work[idx[j]] > work[idx[j - 1]]) { const int t = idx[j]; idx[j] = idx[j - 1]; idx[j - 1] = t; }
  a.order = 0;
  for (int s = 0; s < kMaxProblems; ++s) {
    a.order |= idx[s] << (4 * s);
    a.units[s] = units[idx[s]];
  }
  a.gemm_blocks = a.total;
  args.side.kind = SIDE_NONE;
}

// Adds the side job of a launch whose kernel carries jobs of kind `kind`; returns its workgroups, of `threads` threads.
inline unsigned add_side(KArgs& args, GemmLaunch& g, int kind, int threads) {
  g.side_done = g.side.kind == SIDE_NONE || g.side.kind == kind;
  if (g.side.kind == SIDE_NONE || g.side.kind != kind) return 0;
  args.side = g.side;
  if (kind == SIDE_DGAMMA) return (unsigned)((g.side.d + 31) / 32);
  return (unsigned)((g.side.rows + threads / 64 - 1) / (threads / 64));
}
constexpr int side_kind(bool akc, bool bkc, int epi) {
  return akc == bkc && epi == EPI_GRAD ? SIDE_DGAMMA : akc && !bkc && epi == EPI_STORE ? SIDE_NORM : SIDE_NONE;
}

// The hardware hands consecutive workgroup ids to the 8 XCDs round-robin.  Renumber so
// that each XCD works on one contiguous range of logical ids: neighbouring tiles (which
// share operand panels) then hit the same XCD-private L2.
__device__ inline int xcd_remap(int bid, int nblocks) {
  const int xcd = bid & 7, local = bid >> 3;
  const int q = nblocks >> 3, rem = nblocks & 7;
  return xcd * q + (xcd < rem ? xcd : rem) + local;
}

// 64 bytes of kernel arguments in scalar registers.
typedef __attribute__((ext_vector_type(16))) uint32_t u32x16_t;
typedef const __attribute__((address_space(4))) u32x16_t* KernargPtr;
struct KWords { u32x16_t lo, hi; };

// The head, and a touch of the first problem's lines behind the same wait: the only problem, as often as not, is then a
// hit of the scalar cache.
__device__ inline KHead load_head() {
  KernargPtr k = (KernargPtr)__builtin_amdgcn_kernarg_segment_ptr();
  KWords w = {k[0], k[1]};
  asm volatile("" : "+s"(w.lo), "+s"(w.hi) : "s"(k[2][0]), "s"(k[3][0]));
  return __builtin_bit_cast(KHead, w);
}
__device__ inline KProblem load_problem(int prob) {
  KernargPtr k = (KernargPtr)__builtin_amdgcn_kernarg_segment_ptr();
  KWords w = {k[2 + 2 * prob], k[3 + 2 * prob]};
  asm volatile("" : "+s"(w.lo), "+s"(w.hi));
  return __builtin_bit_cast(KProblem, w);
}

__device__ inline float wave_total(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Gain gradient, 32 columns per workgroup: the threads' 32-column groups share out the rows of sums, and are added in a
// fixed order.  Its own launch takes 4 us behind the norm backward.
template <typename T>
__device__ inline void side_dgamma(const SideJob& j, int block, float* red) {
  const int cl = threadIdx.x & 31, g = threadIdx.x >> 5, groups = blockDim.x >> 5;
  const int c = block * 32 + cl;
  const float* partial = (const float*)j.in;
  float s = 0.f;
  if (c < j.d) {
#pragma unroll 16
    for (int k = g; k < j.nblk; k += groups) s += partial[(int64_t)k * j.d + c];
  }
  red[g * 32 + cl] = s;
  __syncthreads();
  if (g != 0 || c >= j.d) return;
  for (int k = 1; k < groups; ++k) s += red[k * 32 + cl];
  if (j.out_f32) {
    float* o = (float*)j.out;
    o[c] = j.accumulate ? o[c] + s : s;
  } else {
    T* o = (T*)j.out;
    o[c] = (T)(j.accumulate ? (float)o[c] + s : s);
  }
}

// U = norm(H) gamma and rstd, a wave per row, the sums in the order of the kernel that does only this.
template <typename T, int VEC>
__device__ inline void side_norm(const SideJob& j, int block) {
  struct alignas(sizeof(T) * VEC) V { T e[VEC]; };
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)block * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (row >= j.rows) return;
  const T* h = (const T*)j.in + row * j.ld_in;
  T* u = (T*)j.out + row * j.ld_out;
  const int nv = j.d / VEC;
  float ss = 0.f;
#pragma unroll 4
  for (int i = lane; i < nv; i += 64) {
    const V x = *(const V*)(h + i * VEC);
#pragma unroll
    for (int e = 0; e < VEC; ++e) { const float f = (float)x.e[e]; ss += f * f; }
  }
  ss = wave_total(ss);
  const float rs = 1.0f / sqrtf(ss / (float)j.d + j.eps);
  if (lane == 0) j.rstd[row] = rs;
#pragma unroll 4
  for (int i = lane; i < nv; i += 64) {
    const V x = *(const V*)(h + i * VEC), g = *(const V*)((const T*)j.gamma + i * VEC);
    V o;
#pragma unroll
    for (int e = 0; e < VEC; ++e) o.e[e] = (T)((float)x.e[e] * rs * (float)g.e[e]);
    *(V*)(u + i * VEC) = o;
  }
}

// The side job of a workgroup behind those of the products.
template <typename T, int KIND>
__device__ inline void run_side(const KArgs& args, int block, void* smem) {
  if constexpr (KIND == SIDE_DGAMMA) side_dgamma<T>(args.side, block, (float*)smem);
  else if constexpr (KIND == SIDE_NORM) side_norm<T, sizeof(T) == 2 ? 8 : 1>(args.side, block);
}

struct TileCoord { int prob, tm, tn, split, z; };

// The problem of workgroup `bid` and its index there.
__device__ inline int map_problem(const KHead& a, int bid, int* index) {
  const int l = xcd_remap(bid, a.total);
  *index = l;
  if (a.nprob < 2) return 0;      // a single problem: the segments are consecutive eighths of its workgroups
  // Segment x starts at the sum over problems of (x * units) / 8, no later than the first index that xcd_remap gives
  // XCD x: the search for the segment of l goes upward from there.
  auto first = [&](int x) {
    int b = 0;
#pragma unroll
    for (int s = 0; s < kMaxProblems; ++s) b += (x * a.units[s]) >> 3;
    return b;
  };
  int x = bid & 7;
  while (x < 7 && first(x + 1) <= l) ++x;
  int left = l - first(x), prob = 0, t = 0;
#pragma unroll
  for (int s = 0; s < kMaxProblems; ++s) {
    const int b0 = (x * a.units[s]) >> 3, n = (((x + 1) * a.units[s]) >> 3) - b0;
    if (left >= 0 && left < n) { prob = a.order >> (4 * s); t = b0 + left; }
    left -= n;
  }
  *index = __builtin_amdgcn_readfirstlane(t);
  return __builtin_amdgcn_readfirstlane(prob & 15);
}

// Grouped ordering inside one problem: walk GROUP tile-rows together so that concurrently
// running blocks reuse both A panels (same tile-row) and B panels (same tile-column).
template <int BM, int BN>
__device__ inline TileCoord map_tile(const KHead& a, const KProblem& p, int prob, int t) {
  TileCoord tc;
  tc.prob = prob;
  const int tiles_m = (uint32_t)(p.M + BM - 1) / BM, tiles_n = (uint32_t)(p.N + BN - 1) / BN, per = tiles_m * tiles_n;
  const int part = p.splits_kpad >= 4 || a.batch > 1 ? div_by(t, per, p.by_tiles) : 0;
  t -= part * per;
  tc.split = p.splits_kpad >= 4 ? part : 0;    // cut along K: all tiles of one part are consecutive
  tc.z = p.splits_kpad >= 4 ? 0 : part;        // batched products: all tiles of one product are consecutive
  constexpr int GROUP = 8;
  const int gsize = GROUP * tiles_n;
  const int g = div_by(t, gsize, p.by_group);
  const int first_m = g * GROUP, tt = t - g * gsize;
  const int gm = min(tiles_m - first_m, GROUP);
  tc.tn = tt >> 3;
  if (gm < GROUP) {            // the last group, of 1 to 7 tile rows: 65536 / gm rounded up, then corrected
    constexpr uint64_t lo = 0x3334400055568000ull, hi = 0x24932AABull;      // gm = 2 to 5, 6 and 7
    const int m = gm == 1 ? 65536 : (int)((gm < 6 ? lo >> (16 * (gm - 2)) : hi >> (16 * (gm - 6))) & 0xFFFF);
    int q = (int)(((uint64_t)(uint32_t)tt * m) >> 16);
    while (q * gm > tt) --q;
    while ((q + 1) * gm <= tt) ++q;
    tc.tn = q;
  }
  // wave-uniform by construction; told to the compiler so that everything derived from them (buffer offsets, loop
  // bounds) stays in scalar registers
  tc.tn = __builtin_amdgcn_readfirstlane(tc.tn);
  tc.tm = __builtin_amdgcn_readfirstlane(first_m + tt - tc.tn * gm);
  return tc;
}

// A problem as one product of a batch sees it: operand, output and row-vector pointers moved to product z.
// ESZ = bytes per operand / output element.
template <int ESZ>
__device__ inline GemmProblem product_view(const KHead& a, const KProblem& p, int z) {
  GemmProblem q;
#pragma unroll
  for (int s = 0; s < 3; ++s) { q.A[s] = p.A[s]; q.B[s] = p.B[s]; q.C[s] = p.C[s]; }
  q.lda = p.lda; q.ldb = p.ldb; q.ldc = p.ldc;
  q.M = p.M; q.N = p.N; q.K = p.K; q.nseg = p.chunk_nseg & 3; q.chunk = p.chunk_nseg >> 2;
  q.pad_cols = p.aux; q.rope_half = p.aux;
  q.splits = p.splits_kpad >> 1; q.kpad_ok = p.splits_kpad & 1;
  q.rowvec = a.rowvec; q.addend = a.addend; q.scale = a.scale; q.causal = a.causal;
  q.poly_a = a.poly_a; q.poly_b = a.poly_b; q.rope_seq = a.rope_seq;
  q.fold_norm = a.tail != 0;
  if (a.batch > 1) {
    const __attribute__((address_space(4))) int64_t* outer =
        (const __attribute__((address_space(4))) int64_t*)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(KArgs, b_bo) / 8;
    const int zo = __builtin_amdgcn_readfirstlane(z / a.batch_inner), zi = z - zo * a.batch_inner;
    q.A[0] = (const char*)p.A[0] + ((int64_t)zo * a.a_bo + (int64_t)zi * a.a_bi) * ESZ;
    q.B[0] = (const char*)p.B[0] + ((int64_t)zo * outer[0] + (int64_t)zi * a.b_bi) * ESZ;
    q.C[0] = (char*)p.C[0] + ((int64_t)zo * outer[1] + (int64_t)zi * a.c_bi) * ESZ;
    if (a.rowvec) q.rowvec = a.rowvec + (int64_t)z * p.M;
  }
  return q;
}

// Wave-uniform choice between the base pointers of up to three K segments, pinned to scalar
// registers half by half (a select on descriptors is otherwise lowered to per-lane moves and
// every load that uses the result to a loop over lanes).
__device__ inline const void* select_base(int seg, const void* p0, const void* p1, const void* p2) {
  const uint64_t a = (uint64_t)(seg == 0 ? p0 : (seg == 1 ? p1 : p2));
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
  return (const void*)(((uint64_t)hi << 32) | lo);
}

// Softmax products (CAUSAL_TILE): output blocks of 256 x 256 that lie entirely above the diagonal
// are never read by the products that consume the probabilities (their K loops are clipped to the
// same 256-aligned blocks whatever tile size they run with), so tiles inside such a block are
// neither computed nor written.  Tiles above the diagonal but inside a diagonal block still write
// their zeros.  Uniform over the workgroup.
__device__ inline bool causal_tile_unused(const GemmProblem& p, int m0, int n0, int bm) {
  return p.causal == CAUSAL_TILE && (n0 >> 8) > ((m0 + bm - 1) >> 8);
}

// Causal attention products only touch part of K (or nothing): clip the stage range [lo, hi).
__device__ inline void causal_clip(const GemmProblem& p, int m0, int n0, int bm, int bk, int& lo, int& hi) {
  if (p.causal == CAUSAL_NONE) return;
  if (p.causal == CAUSAL_K_FROM_M) lo = max(lo, m0 / bk);
  else if (p.causal == CAUSAL_K_UPTO_M) hi = min(hi, (m0 + bm + bk - 1) / bk);
  else if (p.causal == CAUSAL_TILE && n0 > m0 + bm - 1) hi = lo;
  lo = __builtin_amdgcn_readfirstlane(lo);
  hi = __builtin_amdgcn_readfirstlane(hi);
}

template <typename T> __device__ inline float to_f32(T x) { return (float)x; }
template <typename T> __device__ inline T from_f32(float x) { return (T)x; }

// silu(g) and its derivative.  PRECISE (fp32 storage path) uses expf and a true divide;
// the bf16 path uses the hardware exp2/rcp approximations, far below bf16 resolution.
template <bool PRECISE> __device__ inline float sigmoid_f(float g) {
  if constexpr (PRECISE) {
    return 1.0f / (1.0f + expf(-g));
  } else {
    return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.44269504088896341f * g));
  }
}

template <int EPI> constexpr bool kUnhandledEpilogue = false;

// 1 / sqrt of a squared norm; a zero matrix is left unchanged.
__device__ inline float inv_norm(float sq) { return sq > 0.f ? 1.0f / sqrtf(sq) : 1.0f; }
// From the norms of the kNormBlocks parts of a matrix; every wave for itself, in a fixed order.
__device__ inline float inv_norm_of_parts(const float* norms, int lane) {
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < kNormBlocks / 64; ++i) s += norms[64 * i + lane] * norms[64 * i + lane];
  return inv_norm(wave_total(s));
}
// The norm that the epilogue EPI_HILO divides its result by, through poly_a.
template <int EPI>
__device__ inline void fold_norm(GemmProblem& p, int lane) {
  if (EPI == EPI_HILO) p.poly_a = p.fold_norm ? inv_norm_of_parts(p.rowvec, lane) : 1.f;
}

// One output element (single products) or one (gate, up) pair (dual products).
template <int EPI, typename T>
__device__ inline void epilogue_elem(const GemmProblem& p, const KHead& a, int split,
                                     int row, int col, float v, float v2) {
  if (row >= p.M) return;
  if constexpr (EPI == EPI_STORE) {
    if (col < p.N) {
      const int64_t idx = (int64_t)row * p.ldc + col;
      if (sizeof(T) == 4 || p.splits > 1) ((float*)p.C[0])[(int64_t)split * p.M * p.ldc + idx] = v;
      else ((T*)p.C[0])[idx] = from_f32<T>(v);
    }
  } else if constexpr (EPI == EPI_GRAD) {
    if (col < p.N) {
      const int64_t idx = (int64_t)row * p.ldc + col;
      if (a.out_f32) {
        float* c = (float*)p.C[0];
        c[idx] = a.accumulate ? c[idx] + v : v;
      } else {
        T* c = (T*)p.C[0];
        c[idx] = from_f32<T>(a.accumulate ? to_f32<T>(c[idx]) + v : v);
      }
    }
  } else if constexpr (EPI == EPI_ATTN_P) {
    if (col < p.N) {
      constexpr bool PRECISE = sizeof(T) == 4;
      float pr = 0.f;
      if (col <= row) {
        const float x = v * p.scale - p.rowvec[row];
        pr = PRECISE ? expf(x) : __builtin_amdgcn_exp2f(1.44269504088896341f * x);
      }
      ((T*)p.C[0])[(int64_t)row * p.ldc + col] = from_f32<T>(pr);
    }
  } else if constexpr (EPI == EPI_ATTN_DS) {
    if (col < p.N) {
      T* c = (T*)p.C[0] + (int64_t)row * p.ldc + col;
      *c = from_f32<T>(to_f32<T>(*c) * (v - p.rowvec[row]) * p.scale);
    }
  } else if constexpr (EPI == EPI_RESID) {
    if (col < p.N) {
      const int64_t idx = (int64_t)row * p.ldc + col;
      ((T*)p.C[0])[idx] = from_f32<T>(v + to_f32<T>(((const T*)p.C[1])[idx]));
    }
  } else if constexpr (EPI == EPI_POLY) {
    if (col < p.N) {
      const int64_t idx = (int64_t)row * p.ldc + col;
      float x = p.scale * v;
      if (p.addend) x += p.poly_b * p.addend[idx];
      if (row == col) x += p.poly_a;
      ((T*)p.C[0])[idx] = from_f32<T>(x);
      if (p.C[1]) ((float*)p.C[1])[idx] = v;
    }
  } else if constexpr (EPI == EPI_HILO) {
    if (col < p.N) {
      const int64_t idx = (int64_t)row * p.ldc + col;
      const float y = sizeof(T) == 2 ? v * p.poly_a : v;
      const float x = p.addend ? y + p.addend[idx] : y;
      if (p.C[0]) ((float*)p.C[0])[idx] = x;
      if constexpr (sizeof(T) == 2) {
        const T h = from_f32<T>(x);
        ((T*)p.C[1])[idx] = h;
        if (p.C[2]) ((T*)p.C[2])[idx] = from_f32<T>(x - to_f32<T>(h));
      }
    }
  } else if constexpr (EPI == EPI_SWIGLU_FWD) {
    const int64_t idx = (int64_t)row * p.ldc + col;
    if (col < p.N) {
      constexpr bool PRECISE = sizeof(T) == 4;
      const float sg = sigmoid_f<PRECISE>(v);
      if (p.C[0]) ((T*)p.C[0])[idx] = from_f32<T>(v);
      if (p.C[1]) ((T*)p.C[1])[idx] = from_f32<T>(v2);
      ((T*)p.C[2])[idx] = from_f32<T>(v * sg * v2);
    } else if (col < p.pad_cols) {
      if (p.C[0]) ((T*)p.C[0])[idx] = from_f32<T>(0.f);
      if (p.C[1]) ((T*)p.C[1])[idx] = from_f32<T>(0.f);
      ((T*)p.C[2])[idx] = from_f32<T>(0.f);
    }
  } else if constexpr (EPI == EPI_SWIGLU_BWD) {
    const int64_t idx = (int64_t)row * p.ldc + col;
    T* dg = (T*)p.C[0];
    T* dz = (T*)p.C[1];
    T* aa = (T*)p.C[2];
    if (col < p.N) {
      constexpr bool PRECISE = sizeof(T) == 4;
      const float da = to_f32<T>(dg[idx]);
      const float sg = sigmoid_f<PRECISE>(v);
      const float s = v * sg;
      aa[idx] = from_f32<T>(s * v2);
      dz[idx] = from_f32<T>(da * s);
      dg[idx] = from_f32<T>(da * v2 * (sg * (1.0f + v * (1.0f - sg))));
    } else if (col < p.pad_cols) {
      aa[idx] = from_f32<T>(0.f);
      dz[idx] = from_f32<T>(0.f);
      dg[idx] = from_f32<T>(0.f);
    }
  } else {
    static_assert(kUnhandledEpilogue<EPI>, "no single-element form of this epilogue");
  }
}

constexpr bool epi_is_dual(int epi) { return epi == EPI_SWIGLU_FWD || epi == EPI_SWIGLU_BWD; }

typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4_t;

__device__ inline bf16x4_t pack_bf16x4(float a, float b, float c, float d) {
  bf16x4_t o;
  o[0] = (__bf16)a; o[1] = (__bf16)b; o[2] = (__bf16)c; o[3] = (__bf16)d;
  return o;
}

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8s_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;

__device__ inline bf16x8s_t pack_bf16x8(const float (&v)[8]) {
  bf16x8s_t o;
#pragma unroll
  for (int e = 0; e < 8; ++e) o[e] = (__bf16)v[e];
  return o;
}

// Eight consecutive output columns of one row (bf16 outputs, 16-byte accesses), used by the
// LDS-staged epilogue; falls back to single elements at the ragged right edge.
template <int EPI>
__device__ inline void epilogue_vec8(const GemmProblem& p, const KHead& a, int split, int row, int col0,
                                     const float (&v)[8], const float (&v2)[8]) {
  if (row >= p.M) return;
  if (col0 + 8 > p.N) {
    if constexpr (EPI != EPI_ROPE) {      // whole heads: never ragged
#pragma unroll
      for (int e = 0; e < 8; ++e) epilogue_elem<EPI, __bf16>(p, a, split, row, col0 + e, v[e], v2[e]);
    }
    return;
  }
  const int64_t idx = (int64_t)row * p.ldc + col0;
  if constexpr (EPI == EPI_STORE) {
    *(bf16x8s_t*)((__bf16*)p.C[0] + idx) = pack_bf16x8(v);
  } else if constexpr (EPI == EPI_ATTN_P) {
    const float lse = p.rowvec[row];
    float o[8];
#pragma unroll
    for (int e = 0; e < 8; ++e)
      o[e] = (col0 + e <= row) ? __builtin_amdgcn_exp2f(1.44269504088896341f * (v[e] * p.scale - lse)) : 0.f;
    *(bf16x8s_t*)((__bf16*)p.C[0] + idx) = pack_bf16x8(o);
  } else if constexpr (EPI == EPI_ATTN_DS) {
    bf16x8s_t* c = (bf16x8s_t*)((__bf16*)p.C[0] + idx);
    const bf16x8s_t pr = *c;
    const float dsum = p.rowvec[row];
    float o[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = (float)pr[e] * (v[e] - dsum) * p.scale;
    *c = pack_bf16x8(o);
  } else if constexpr (EPI == EPI_GRAD) {      // bf16 gradients; fp32 ones take epilogue_vec4
    bf16x8s_t* c = (bf16x8s_t*)((__bf16*)p.C[0] + idx);
    float o[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = v[e];
    if (a.accumulate) {
      const bf16x8s_t old = *c;
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] += (float)old[e];
    }
    *c = pack_bf16x8(o);
  } else if constexpr (EPI == EPI_RESID) {
    const bf16x8s_t r = *(const bf16x8s_t*)((const __bf16*)p.C[1] + idx);
    float o[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = v[e] + (float)r[e];
    *(bf16x8s_t*)((__bf16*)p.C[0] + idx) = pack_bf16x8(o);
  } else if constexpr (EPI == EPI_ROPE) {      // v2: the partner columns
    float o[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = v[e];
    if (p.rope_half) {
      const int64_t at = (int64_t)(row % p.rope_seq) * p.rope_half + (col0 & (p.rope_half - 1));
      const float sgn = (col0 & p.rope_half) ? 1.f : -1.f;
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const f32x4_t c = *(const f32x4_t*)(p.rowvec + at + 4 * q), s = *(const f32x4_t*)(p.addend + at + 4 * q);
#pragma unroll
        for (int e = 0; e < 4; ++e) o[4 * q + e] = v[4 * q + e] * c[e] + sgn * v2[4 * q + e] * s[e];
      }
    }
    *(bf16x8s_t*)((__bf16*)p.C[0] + idx) = pack_bf16x8(o);
  } else if constexpr (EPI == EPI_POLY) {
    float o[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = p.scale * v[e];
    if (p.addend) {
      const f32x4_t r0 = *(const f32x4_t*)(p.addend + idx), r1 = *(const f32x4_t*)(p.addend + idx + 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) { o[e] += p.poly_b * r0[e]; o[4 + e] += p.poly_b * r1[e]; }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if (row == col0 + e) o[e] += p.poly_a;
    *(bf16x8s_t*)((__bf16*)p.C[0] + idx) = pack_bf16x8(o);
    if (p.C[1]) {
      float* raw = (float*)p.C[1] + idx;
      const f32x4_t o0 = {v[0], v[1], v[2], v[3]}, o1 = {v[4], v[5], v[6], v[7]};
      *(f32x4_t*)raw = o0;
      *(f32x4_t*)(raw + 4) = o1;
    }
  } else if constexpr (EPI == EPI_SWIGLU_FWD) {
    float av[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) av[e] = v[e] * sigmoid_f<false>(v[e]) * v2[e];
    if (p.C[0]) *(bf16x8s_t*)((__bf16*)p.C[0] + idx) = pack_bf16x8(v);
    if (p.C[1]) *(bf16x8s_t*)((__bf16*)p.C[1] + idx) = pack_bf16x8(v2);
    *(bf16x8s_t*)((__bf16*)p.C[2] + idx) = pack_bf16x8(av);
  } else if constexpr (EPI == EPI_SWIGLU_BWD) {
    bf16x8s_t* dg = (bf16x8s_t*)((__bf16*)p.C[0] + idx);
    const bf16x8s_t da8 = *dg;
    float oa[8], oz[8], og[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float da = (float)da8[e];
      const float sg = sigmoid_f<false>(v[e]);
      const float s = v[e] * sg;
      oa[e] = s * v2[e];
      oz[e] = da * s;
      og[e] = da * v2[e] * (sg * (1.0f + v[e] * (1.0f - sg)));
    }
    *(bf16x8s_t*)((__bf16*)p.C[2] + idx) = pack_bf16x8(oa);
    *(bf16x8s_t*)((__bf16*)p.C[1] + idx) = pack_bf16x8(oz);
    *dg = pack_bf16x8(og);
  } else {
    static_assert(kUnhandledEpilogue<EPI>, "no eight-column form of this epilogue");
  }
}

// Four consecutive output columns of one row (fp32 outputs, 16-byte stores; bf16 gradients of the register-staged
// kernel) when the group lies inside the matrix, else element by element.  Row strides are multiples of 8
// elements and col0 of 4, so the vector accesses are aligned.
template <int EPI>
__device__ inline void epilogue_vec4(const GemmProblem& p, const KHead& a, int split, int row, int col0,
                                     const float (&v)[4]) {
  if (row >= p.M) return;
  if (col0 + 4 > p.N) {
#pragma unroll
    for (int e = 0; e < 4; ++e) epilogue_elem<EPI, __bf16>(p, a, split, row, col0 + e, v[e], 0.f);
    return;
  }
  const int64_t idx = (int64_t)row * p.ldc + col0;
  if constexpr (EPI == EPI_STORE) {            // a part of a product that is cut along K
    f32x4_t o = {v[0], v[1], v[2], v[3]};
    *(f32x4_t*)((float*)p.C[0] + (int64_t)split * p.M * p.ldc + idx) = o;
  } else if constexpr (EPI == EPI_GRAD) {
    if (a.out_f32) {
      f32x4_t* c = (f32x4_t*)((float*)p.C[0] + idx);
      f32x4_t o = {v[0], v[1], v[2], v[3]};
      if (a.accumulate) o += *c;
      *c = o;
    } else {
      bf16x4_t* c = (bf16x4_t*)((__bf16*)p.C[0] + idx);
      if (a.accumulate) {
        const bf16x4_t old = *c;
        *c = pack_bf16x4(v[0] + (float)old[0], v[1] + (float)old[1], v[2] + (float)old[2], v[3] + (float)old[3]);
      } else {
        *c = pack_bf16x4(v[0], v[1], v[2], v[3]);
      }
    }
  } else if constexpr (EPI == EPI_HILO) {
    f32x4_t x = {v[0], v[1], v[2], v[3]};
    x *= p.poly_a;
    if (p.addend) x += *(const f32x4_t*)(p.addend + idx);
    if (p.C[0]) *(f32x4_t*)((float*)p.C[0] + idx) = x;
    const bf16x4_t h = pack_bf16x4(x[0], x[1], x[2], x[3]);
    *(bf16x4_t*)((__bf16*)p.C[1] + idx) = h;
    if (p.C[2])
      *(bf16x4_t*)((__bf16*)p.C[2] + idx) =
          pack_bf16x4(x[0] - (float)h[0], x[1] - (float)h[1], x[2] - (float)h[2], x[3] - (float)h[3]);
  } else {
    static_assert(kUnhandledEpilogue<EPI>, "no four-column form of this epilogue");
  }
}

}  // namespace mecefo
