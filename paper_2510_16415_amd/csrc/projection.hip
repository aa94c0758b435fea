// Projection refresh of Alg. 3: an orthonormal basis of (an approximation to) the span of the
// top-r right (or left) singular vectors of a weight matrix, computed without an SVD or a QR:
// subspace iteration X <- W^T (W X) on the GEMM core, with Newton-Schulz steps X <- X q(X^T X)
// in between.  A right-multiplication by an invertible r x r matrix changes the basis but not its
// span, so the Newton-Schulz steps only control the conditioning of the basis (they push every
// singular value of X towards 1); the final steps use the form X + X E, E = (I - X^T X)/2, whose
// small correction keeps full relative precision in the storage type.
#include <math.h>
#include <string.h>

#include "../../include/mecefo.h"
#include "gemm_bf16_launch.hip.h"
#include "mecefo_internal.h"

namespace mecefo {
namespace {

constexpr int kHeldSplits = 8;

// For fp32 weights the iterate is one fp32 matrix.  For bf16 weights it enters the MFMA products as the
// sum of two bf16 matrices (hi = bf16(x), lo = bf16(x - hi): 16 mantissa bits), contracted as two K
// segments of one launch: a single bf16 rounding of the iterate would drown the weakest of the r
// directions, whose share of X after one application of W^T W is (s_r/s_1)^2.  The halves are written by
// whatever produces the iterate: the product's epilogue, the sum of its K splits, the normalisation.  An fp32 copy is
// written where something reads it: the result of a power round (normalised next), of a step in front of a polishing step
// (which adds to it) and of the last step unless that writes P itself.
//
// A refresh is a chain of some 60 dependent products of a few microseconds each, so launches count: with
// the polynomial and the halves in the epilogues a Newton-Schulz step is three products (four launches where
// the Gram matrix is cut along K) instead of three products, two or three elementwise kernels and a copy.
// Three matrices of [5461 x 2048], rank 512, two rounds of eight steps and three polishing steps: 406 launches and
// 6760 us on the register-staged kernels with separate elementwise launches, 218 and 1970 us now (3390 -> 2650 us by the
// epilogues alone).

// Sum of the K splits of a product, finished like its epilogue would (EPI_POLY or EPI_HILO; fixed order).
struct SplitSum {
  const float* partial;
  int splits;
  int64_t mn, ld;          // elements and row stride of one part
  float* raw;              // fp32 result (EPI_POLY: the plain sum), may be NULL
  __bf16 *hi, *lo;         // EPI_HILO: the two halves; EPI_POLY: hi is the polynomial
  const float* addend;
  float a, b, c;           // EPI_POLY
  const float* norm;       // EPI_HILO: the norms of the parts of the matrix whose norm it divides by, or NULL
};
template <int EPI>
__global__ __launch_bounds__(256) void split_sum_kernel(const SplitSum q) {
  float k = 1.f;
  if (EPI == EPI_HILO && q.norm) k = inv_norm_of_parts(q.norm, threadIdx.x & 63);
  const int64_t i4 = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;     // mn is a multiple of 8
  if (i4 >= q.mn) return;
  typedef __attribute__((ext_vector_type(4))) float f4;
  typedef __attribute__((ext_vector_type(4))) __bf16 h4;
  f4 s = *(const f4*)(q.partial + i4);
#pragma unroll 4
  for (int j = 1; j < q.splits; ++j) s += *(const f4*)(q.partial + (int64_t)j * q.mn + i4);
  h4 h, l;
  if constexpr (EPI == EPI_POLY) {
    if (q.raw) *(f4*)(q.raw + i4) = s;
    f4 x = s * q.c;
    if (q.addend) x += *(const f4*)(q.addend + i4) * q.b;
    const int64_t row = i4 / q.ld, col = i4 - row * q.ld;                // four columns of one row: ld % 8 == 0
#pragma unroll
    for (int e = 0; e < 4; ++e) h[e] = (__bf16)(col + e == row ? x[e] + q.a : x[e]);
    *(h4*)(q.hi + i4) = h;
  } else {
    s *= k;
    if (q.addend) s += *(const f4*)(q.addend + i4);
    if (q.raw) *(f4*)(q.raw + i4) = s;
#pragma unroll
    for (int e = 0; e < 4; ++e) { h[e] = (__bf16)s[e]; l[e] = (__bf16)(s[e] - (float)h[e]); }
    *(h4*)(q.hi + i4) = h;
    if (q.lo) *(h4*)(q.lo + i4) = l;
  }
}

// The Frobenius norm of the part of X that a block has, in norms[block].  Block b sums rows b, b + gridDim.x, ... in a
// fixed order, thread t the groups of four columns t, t + 256, ... and the rows four at a time, so that four loads are in
// flight (one scalar load after another: 8.5 us for [5461 x 512]; the refresh with nine of them went from 2435 to 2377 us).
// The squares are summed in 64 bits: those of W^T W X are fourth powers of W's scale, which leave fp32's range for weights
// below 1e-10 and above 1e9; the norms themselves are as far inside it as X is.
template <typename T>
__global__ __launch_bounds__(256) void norm_parts_kernel(const T* __restrict__ X, int64_t ld, int64_t rows,
                                                         int cols, float* __restrict__ norms) {
  __shared__ double red[256];
  typedef __attribute__((ext_vector_type(4))) T t4;
  // columns [cols, ld) hold anything: groups of four that reach behind `cols` are cut off element by element
  const int groups = (cols + 3) / 4;
  // a block row is wide enough for `lanes` groups; the other threads take further rows of the block
  const int lanes = groups < 256 ? groups : 256, per = 256 / lanes;
  const int sub = threadIdx.x / lanes, lane = threadIdx.x - sub * lanes;
  double acc = 0.0;
  if (sub < per) {
    const int64_t step = (int64_t)gridDim.x * per;
    for (int64_t row0 = (int64_t)blockIdx.x * per + sub; row0 < rows; row0 += 4 * step)
      for (int g = lane; g < groups; g += lanes) {
        t4 v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int64_t row = row0 + q * step < rows ? row0 + q * step : row0;
          v[q] = *(const t4*)(X + row * ld + 4 * g);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (row0 + q * step < rows) {
#pragma unroll
            for (int e = 0; e < 4; ++e) acc += 4 * g + e < cols ? (double)(float)v[q][e] * (double)(float)v[q][e] : 0.0;
          }
      }
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) norms[blockIdx.x] = (float)sqrt(red[0]);
}

// X / |X| from the norms of its parts; a zero matrix is left unchanged.  Every block adds the kNormBlocks squares by
// itself, as a tree over its threads (one thread adding them one by one took 12 to 20 us).  The result goes back to X
// (keep) and, with hi, out as halves (X is a multiple of four elements: padded rows).
__global__ __launch_bounds__(256) void scale_by_inv_norm_kernel(float* __restrict__ X, int64_t n,
                                                                const float* __restrict__ norms, bool keep,
                                                                __bf16* __restrict__ hi, __bf16* __restrict__ lo) {
  __shared__ double red[256];
  static_assert(kNormBlocks == 256, "one norm per thread");
  red[threadIdx.x] = (double)norms[threadIdx.x] * (double)norms[threadIdx.x];
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  const float k = red[0] > 0.0 ? (float)(1.0 / sqrt(red[0])) : 1.f;
  typedef __attribute__((ext_vector_type(4))) float f4;
  typedef __attribute__((ext_vector_type(4))) __bf16 h4;
  for (int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4; i < n; i += (int64_t)gridDim.x * 1024) {
    const f4 x = *(const f4*)(X + i) * k;
    if (keep) *(f4*)(X + i) = x;
    if (!hi) continue;
    h4 h, l;
#pragma unroll
    for (int e = 0; e < 4; ++e) { h[e] = (__bf16)x[e]; l[e] = (__bf16)(x[e] - (float)h[e]); }
    *(h4*)(hi + i) = h;
    *(h4*)(lo + i) = l;
  }
}

// dst[rows x cols] (row stride ldd) = src (row stride lds), converting the element type;
// columns [cols, ldd_fill) of dst are set to zero.
template <typename D, typename S>
__global__ __launch_bounds__(256) void convert2d_kernel(D* __restrict__ dst, int64_t ldd, const S* __restrict__ src,
                                                        int64_t lds, int64_t rows, int cols, int fill_to) {
  const int64_t n = rows * fill_to;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const int64_t row = i / fill_to;
    const int c = (int)(i - row * fill_to);
    dst[row * ldd + c] = c < cols ? (D)(float)src[row * lds + c] : (D)0.f;
  }
}

inline int64_t up(int64_t x, int64_t a) { return (x + a - 1) / a * a; }
inline unsigned grid_for(int64_t n) { int64_t g = (n + 255) / 256; return (unsigned)(g < 1 ? 1 : (g > 65536 ? 65536 : g)); }

struct Plan {
  bool bf16;
  int esz;
  int m, n, r;       // W is [m x n]; the basis has `dim` rows (n for right, m for left vectors)
  int dim, other;
  int64_t ldx;       // row stride of every internal [* x r] buffer
  size_t X32[2], Y32, Xh[2], Xl[2], Yh, Yl, A32, M16, A16, part, partial, total;
};

Plan make_plan(bool bf16, int m, int n, int r, int left) {
  Plan p;
  p.bf16 = bf16; p.esz = bf16 ? 2 : 4;
  p.m = m; p.n = n; p.r = r;
  p.dim = left ? m : n; p.other = left ? n : m;
  p.ldx = up(r, 8);
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off += (size_t)up((int64_t)bytes, 256); return o; };
  p.X32[0] = take((size_t)p.dim * p.ldx * 4);
  p.X32[1] = take((size_t)p.dim * p.ldx * 4);
  p.Y32 = take((size_t)p.other * p.ldx * 4);
  const size_t hx = bf16 ? (size_t)p.dim * p.ldx * 2 : 0, hy = bf16 ? (size_t)p.other * p.ldx * 2 : 0;
  // bf16: a step updates the one fp32 master copy in place while its product still reads the halves, so the
  // halves take turns; the second pair lies where fp32 keeps its second copy.  fp32: X32 takes turns.
  p.Xh[0] = take(hx); p.Xl[0] = take(hx);
  p.Xh[1] = p.X32[1]; p.Xl[1] = p.X32[1] + hx;
  p.Yh = take(hy); p.Yl = take(hy);
  p.A32 = take((size_t)r * p.ldx * 4);
  p.M16 = take((size_t)r * p.ldx * p.esz);
  p.A16 = take((size_t)r * p.ldx * p.esz);
  p.part = take(kNormBlocks * 4);
  // split-K partials of the products with few output tiles and a long contraction
  const int64_t big = (p.dim > p.other ? p.dim : p.other);
  p.partial = take(bf16 ? (size_t)kHeldSplits * big * p.ldx * 4 : 0);
  p.total = off + 256;
  return p;
}

// An iterate as GEMM operand: fp32 path: the master copy; bf16 path: the hi and lo halves.
struct Operand { const void* hi; const void* lo; };

// C (fp32, row stride ldx) = opA * opB, where exactly one of the two sides may be an iterate
// split into hi + lo (then the launch has two K segments over the same other operand).
GemmLaunch product(const Plan& pl, bool akc, bool bkc, const void* A_hi, const void* A_lo, int64_t lda,
                   const void* B_hi, const void* B_lo, int64_t ldb, float* C, int M, int N, int K) {
  GemmLaunch g;
  memset(&g, 0, sizeof(g));
  g.a_kcontig = akc; g.b_kcontig = bkc; g.epi = EPI_GRAD; g.bf16 = pl.bf16; g.out_f32 = true;
  g.nprob = 1;
  GemmProblem& p = g.p[0];
  const bool two = A_lo != nullptr || B_lo != nullptr;
  p.A[0] = A_hi; p.A[1] = A_lo ? A_lo : A_hi; p.A[2] = A_hi;
  p.B[0] = B_hi; p.B[1] = B_lo ? B_lo : B_hi; p.B[2] = B_hi;
  p.C[0] = C;
  p.lda = lda; p.ldb = ldb; p.ldc = pl.ldx; p.M = M; p.N = N; p.K = K; p.nseg = two ? 2 : 1;
  return g;
}

// Products with few output tiles and a long contraction are cut along K when that pays for summing the
// fp32 partials (in a fixed order), into no more parts than the plan's partial buffer holds.
hipError_t run_product(const Plan& pl, char* base, GemmLaunch& g, hipStream_t s) {
  GemmProblem& p = g.p[0];
  int splits = 1;
  if (pl.bf16) {
    bf16_plan_splits(g, (int64_t)kHeldSplits * (pl.dim > pl.other ? pl.dim : pl.other) * pl.ldx);
    splits = p.splits;
    p.splits = 1;
  }
  if (splits <= 1) return launch_gemm(g, s);
  const int epi = g.epi;
  GemmLaunch cut = g;
  float* const partial = (float*)(base + pl.partial);
  cut.epi = EPI_STORE;
  cut.p[0].splits = splits;
  cut.p[0].C[0] = partial;
  hipError_t e = launch_gemm(cut, s);
  if (e != hipSuccess) return e;
  const int64_t mn = (int64_t)p.M * p.ldc;
  if (epi == EPI_GRAD) {
    const SumJob job{partial, p.C[0], mn, splits};
    return launch_sum_parts(false, &job, 1, s);
  }
  const dim3 grid((unsigned)((mn + 1023) / 1024));
  SplitSum q{partial, splits, mn, p.ldc, nullptr, nullptr, nullptr, p.addend, p.poly_a, p.poly_b, p.scale,
             p.fold_norm ? p.rowvec : nullptr};
  if (epi == EPI_POLY) {
    q.raw = (float*)p.C[1]; q.hi = (__bf16*)p.C[0];
    hipLaunchKernelGGL(split_sum_kernel<EPI_POLY>, grid, dim3(256), 0, s, q);
  } else {
    q.raw = (float*)p.C[0]; q.hi = (__bf16*)p.C[1]; q.lo = (__bf16*)p.C[2];
    hipLaunchKernelGGL(split_sum_kernel<EPI_HILO>, grid, dim3(256), 0, s, q);
  }
  return hipGetLastError();
}

#define HIP_TRY(x) do { hipError_t e__ = (x); if (e__ != hipSuccess) return (mecefo_status_t)fail(MECEFO_ERR_LAUNCH, "%s: %s", #x, hipGetErrorString(e__)); } while (0)

struct Refresh {
  Plan pl;
  char* base;
  hipStream_t s;
  int cur = 0;

  // `cur` says which copy holds the iterate: of X32 (fp32 path) or of its halves (bf16 path, X32 is one).
  float* X32() const { return (float*)(base + pl.X32[pl.bf16 ? 0 : cur]); }
  float* X32_next() const { return (float*)(base + pl.X32[pl.bf16 ? 0 : cur ^ 1]); }
  float* Y32() const { return (float*)(base + pl.Y32); }
  Operand opX() const { return pl.bf16 ? Operand{base + pl.Xh[cur], base + pl.Xl[cur]} : Operand{X32(), nullptr}; }
  Operand opY() const { return pl.bf16 ? Operand{base + pl.Yh, base + pl.Yl} : Operand{Y32(), nullptr}; }
  // the product's result as an iterate: fp32 `x32` and, bf16 path, its halves
  void to_iterate(GemmLaunch& g, float* x32, size_t hi, size_t lo, const float* addend) const {
    g.epi = EPI_HILO;
    g.p[0].C[0] = x32;
    g.p[0].C[1] = pl.bf16 ? base + hi : nullptr;
    g.p[0].C[2] = pl.bf16 ? base + lo : nullptr;
    g.p[0].addend = addend;
  }
  static void to_poly(GemmLaunch& g, void* out, float* raw, const float* addend, float a, float b, float c) {
    g.epi = EPI_POLY;
    g.p[0].C[0] = out; g.p[0].C[1] = raw;
    g.p[0].addend = addend; g.p[0].poly_a = a; g.p[0].poly_b = b; g.p[0].scale = c;
  }

  // X /= ||X||_F, so that every singular value is <= 1.  keep32: the bf16 path keeps the fp32 copy as well as the halves
  hipError_t normalise(bool keep32) const {
    float* part = (float*)(base + pl.part);
    const int64_t n = (int64_t)pl.dim * pl.ldx;
    hipLaunchKernelGGL(norm_parts_kernel<float>, dim3(kNormBlocks), dim3(256), 0, s, X32(), pl.ldx, (int64_t)pl.dim, pl.r, part);
    hipLaunchKernelGGL(scale_by_inv_norm_kernel, dim3((unsigned)(n < 1024 * 1024 ? (n + 1023) / 1024 : 1024)), dim3(256), 0, s, X32(), n, part,
                       keep32 || !pl.bf16,
                       (__bf16*)(pl.bf16 ? base + pl.Xh[cur] : nullptr), (__bf16*)(pl.bf16 ? base + pl.Xl[cur] : nullptr));
    return hipGetLastError();
  }

  // One Newton-Schulz step X <- X (a I + b A + c A^2), A = X^T X; `additive` (c == 0): X <- X + X E
  // with E = (a - 1) I + b A.  A, A^2 and the polynomial only shape the conditioning and are taken
  // in the storage type; the product with X keeps the split operand.  The fp32 copy of the result is written when it
  // will be read (keep32).  out: where the bf16 half hi goes instead of the workspace (the result's last step).
  mecefo_status_t ns_step(float a, float b, float c, bool additive, bool keep32, void* out) {
    const int r = pl.r, dim = pl.dim;
    float* A32 = (float*)(base + pl.A32);
    void* M16 = base + pl.M16;
    void* A16 = pl.bf16 ? base + pl.A16 : (void*)A32;     // A in the storage type
    const Operand x = opX();
    {  // A = X^T X  [r x r], contraction over the rows of X (hi part only)
      GemmLaunch g = product(pl, false, false, x.hi, nullptr, pl.ldx, x.hi, nullptr, pl.ldx, nullptr, r, r, dim);
      if (additive) to_poly(g, M16, nullptr, nullptr, a - 1.f, 0.f, b);
      else to_poly(g, A16, pl.bf16 ? A32 : nullptr, nullptr, 0.f, 0.f, 1.f);
      HIP_TRY(run_product(pl, base, g, s));
    }
    if (!additive) {  // a I + b A + c A^2, A^2 = A A^T (A is symmetric)
      GemmLaunch g = product(pl, true, true, A16, nullptr, pl.ldx, A16, nullptr, pl.ldx, nullptr, r, r, r);
      to_poly(g, M16, nullptr, A32, a, b, c);
      HIP_TRY(run_product(pl, base, g, s));
    }
    // the polynomial of the symmetric A is symmetric: X M = X M^T, so M is the K-contiguous operand
    GemmLaunch g = product(pl, true, true, x.hi, x.lo, pl.ldx, M16, nullptr, pl.ldx, nullptr, dim, r, r);
    to_iterate(g, keep32 || !pl.bf16 ? X32_next() : nullptr, pl.Xh[cur ^ 1], pl.Xl[cur ^ 1], additive ? X32() : nullptr);
    if (out) { g.p[0].C[1] = out; g.p[0].C[2] = nullptr; }
    HIP_TRY(run_product(pl, base, g, s));
    cur ^= 1;
    return MECEFO_OK;
  }

  // Quintic steps with slope 3.4445 at zero: a small singular value grows by that factor per step,
  // values near 1 stay within about [0.7, 1.2] (the odd quintic used for low-precision
  // orthogonalisation; it does not converge to exactly 1, the cubic steps do).
  mecefo_status_t condition(int steps, bool keep32, void* out) {
    for (int i = 0; i < steps; ++i) {
      const bool last = i == steps - 1;
      mecefo_status_t e = ns_step(3.4445f, -4.7750f, 2.0315f, false, last && keep32, last ? out : nullptr);
      if (e != MECEFO_OK) return e;
    }
    return MECEFO_OK;
  }

  // X <- W^T (W X), in fp32, to be normalised next.  start: the start basis in the caller's memory (bf16), which Y takes
  // over 1 / its norm (`part` holds the norms of its parts), else NULL.
  mecefo_status_t power_round(const void* W, int64_t ldw, int left, const void* start, int64_t ldstart) {
    const int m = pl.m, n = pl.n, r = pl.r;
    const Operand x = start ? Operand{start, nullptr} : opX();
    const int64_t ldx = start ? ldstart : pl.ldx;
    // right vectors: Y = W X [m x r] (K = n), X' = W^T Y [n x r] (K = m, W read as [K x M]);
    // left vectors:  Y = W^T X [n x r] (K = m), X' = W Y [m x r] (K = n)
    GemmLaunch g1 = left ? product(pl, false, false, W, nullptr, ldw, x.hi, x.lo, ldx, nullptr, n, r, m)
                         : product(pl, true, false, W, nullptr, ldw, x.hi, x.lo, ldx, nullptr, m, r, n);
    to_iterate(g1, pl.bf16 ? nullptr : Y32(), pl.Yh, pl.Yl, nullptr);
    if (start) { g1.p[0].fold_norm = true; g1.p[0].rowvec = (const float*)(base + pl.part); }
    HIP_TRY(run_product(pl, base, g1, s));
    const Operand y = opY();
    GemmLaunch g2 = left ? product(pl, true, false, W, nullptr, ldw, y.hi, y.lo, pl.ldx, X32_next(), m, r, n)
                         : product(pl, false, false, W, nullptr, ldw, y.hi, y.lo, pl.ldx, X32_next(), n, r, m);
    HIP_TRY(run_product(pl, base, g2, s));
    cur ^= 1;
    return MECEFO_OK;
  }
};

mecefo_status_t check(int m, int n, int64_t ldw, int r, mecefo_dtype_t dtype, int power_iters, int cond_steps,
                      int polish_steps, bool* bf16) {
  if (dtype != MECEFO_F32 && dtype != MECEFO_BF16) return (mecefo_status_t)fail(MECEFO_ERR_INVALID_ARG, "dtype must be MECEFO_F32 or MECEFO_BF16");
  *bf16 = dtype == MECEFO_BF16;
  if (m < 1 || n < 1) return (mecefo_status_t)fail(MECEFO_ERR_INVALID_ARG, "m >= 1 and n >= 1 required");
  if (r < 1 || r > (m < n ? m : n)) return (mecefo_status_t)fail(MECEFO_ERR_INVALID_ARG, "rank %d outside [1, min(m, n) = %d]", r, m < n ? m : n);
  if (ldw < n) return (mecefo_status_t)fail(MECEFO_ERR_INVALID_ARG, "ldw %lld < n %d", (long long)ldw, n);
  if (*bf16 && ldw % 8) return (mecefo_status_t)fail(MECEFO_ERR_INVALID_ARG, "bf16 path needs ldw to be a multiple of 8");
  if ((int64_t)m * ldw * 4 >= ((int64_t)1 << 31) || (int64_t)(m > n ? m : n) * up(r, 8) * 4 >= ((int64_t)1 << 31))
    return (mecefo_status_t)fail(MECEFO_ERR_UNSUPPORTED, "the matrix or the basis reaches 2 GiB");
  if (power_iters < 0 || cond_steps < 0 || polish_steps < 0 || power_iters > 1000 || cond_steps > 100 || polish_steps > 100)
    return (mecefo_status_t)fail(MECEFO_ERR_INVALID_ARG, "iteration counts must be non-negative (and sane)");
  return MECEFO_OK;
}

}  // namespace
}  // namespace mecefo

using namespace mecefo;

extern "C" {

mecefo_status_t mecefo_projection_workspace_bytes(mecefo_dtype_t dtype, int m, int n, int r, int left,
                                                  size_t* out_bytes) {
  bool bf16;
  mecefo_status_t st = check(m, n, (n + 7) / 8 * 8, r, dtype, 0, 0, 0, &bf16);
  if (st != MECEFO_OK) return st;
  if (!out_bytes) return (mecefo_status_t)fail(MECEFO_ERR_INVALID_ARG, "out_bytes is NULL");
  *out_bytes = make_plan(bf16, m, n, r, left).total;
  return MECEFO_OK;
}

mecefo_status_t mecefo_projection_refresh(mecefo_dtype_t dtype, const void* W, int m, int n, int64_t ldw, int left,
                                          const void* V0, int64_t ldv, int r, int power_iters, int cond_steps,
                                          int polish_steps, void* P, int64_t ldp, void* ws, size_t ws_bytes,
                                          void* hip_stream) {
  bool bf16;
  mecefo_status_t st = check(m, n, ldw, r, dtype, power_iters, cond_steps, polish_steps, &bf16);
  if (st != MECEFO_OK) return st;
  if (!W || !V0 || !P) return (mecefo_status_t)fail(MECEFO_ERR_INVALID_ARG, "W, V0 and P are required");
  if (ldv < r || ldp < r) return (mecefo_status_t)fail(MECEFO_ERR_INVALID_ARG, "ldv and ldp must be >= r");
  const int al = bf16 ? 16 : 4;
  if (((uintptr_t)W | (uintptr_t)V0 | (uintptr_t)P) % al) return (mecefo_status_t)fail(MECEFO_ERR_INVALID_ARG, "W, V0 and P must be %d-byte aligned", al);
  Refresh R;
  R.pl = make_plan(bf16, m, n, r, left);
  if (R.pl.total > ws_bytes) return (mecefo_status_t)fail(MECEFO_ERR_WORKSPACE_TOO_SMALL, "workspace has %zu bytes, %zu needed", ws_bytes, R.pl.total);
  if (!ws) return (mecefo_status_t)fail(MECEFO_ERR_INVALID_ARG, "workspace is NULL");
  R.base = (char*)up((int64_t)(uintptr_t)ws, 256);
  R.s = (hipStream_t)hip_stream;
  const Plan& pl = R.pl;
  const int dim = pl.dim;
  const int64_t ldx = pl.ldx;
  const unsigned gx = grid_for((int64_t)dim * ldx);

  // bf16: the start basis is an operand of the first product where it lies (its rows keep 16-byte alignment, and the
  // product's 32-bit offsets reach all of them), and the last step writes P where its rows have no padding.
  const bool reached = dim == 1 || ldv <= (0x7FFFFFFF / 2 - r) / (dim - 1);
  const bool direct = bf16 && power_iters > 0 && ldv % 8 == 0 && reached;
  void* const out = bf16 && ldp == ldx && r == ldx && (polish_steps > 0 || cond_steps > 0) ? P : nullptr;
  if (direct) {
    hipLaunchKernelGGL(norm_parts_kernel<__bf16>, dim3(kNormBlocks), dim3(256), 0, R.s, (const __bf16*)V0, ldv, (int64_t)dim, r, (float*)(R.base + pl.part));
    HIP_TRY(hipGetLastError());
  } else {
    // start basis -> fp32 master copy (padding columns zeroed: they are contracted as K padding)
    if (bf16) hipLaunchKernelGGL((convert2d_kernel<float, __bf16>), dim3(gx), dim3(256), 0, R.s, R.X32(), ldx, (const __bf16*)V0, ldv, (int64_t)dim, r, (int)ldx);
    else hipLaunchKernelGGL((convert2d_kernel<float, float>), dim3(gx), dim3(256), 0, R.s, R.X32(), ldx, (const float*)V0, ldv, (int64_t)dim, r, (int)ldx);
    HIP_TRY(hipGetLastError());
    HIP_TRY(R.normalise(power_iters == 0 && cond_steps == 0));
  }
  // The start basis is only normalised: a previous projection is orthonormal already and Gaussian
  // noise is well conditioned; without power rounds it is conditioned for the polishing steps.
  if (power_iters == 0) {
    st = R.condition(cond_steps, polish_steps > 0 || !out, polish_steps == 0 ? out : nullptr);
    if (st != MECEFO_OK) return st;
  }
  for (int it = 0; it < power_iters; ++it) {
    const bool last = it == power_iters - 1;
    st = R.power_round(W, ldw, left, direct && it == 0 ? V0 : nullptr, ldv);
    if (st != MECEFO_OK) return st;
    // Before it is split into halves and multiplied with itself: squares and fifth powers of its scale, which is that of
    // W^T W, would leave fp32's range.  The fp32 copy is read by a first polishing step and by the conversion to P.
    HIP_TRY(R.normalise(last && cond_steps == 0));
    st = R.condition(cond_steps, last && (polish_steps > 0 || !out), last && polish_steps == 0 ? out : nullptr);
    if (st != MECEFO_OK) return st;
  }
  for (int i = 0; i < polish_steps; ++i) {  // cubic steps X <- X + X (I - X^T X) / 2
    const bool last = i == polish_steps - 1;
    st = R.ns_step(1.5f, -0.5f, 0.f, true, !last || !out, last ? out : nullptr);
    if (st != MECEFO_OK) return st;
  }
  if (out) return MECEFO_OK;
  const unsigned gp = grid_for((int64_t)dim * r);
  if (bf16) hipLaunchKernelGGL((convert2d_kernel<__bf16, float>), dim3(gp), dim3(256), 0, R.s, (__bf16*)P, ldp, R.X32(), ldx, (int64_t)dim, r, r);
  else hipLaunchKernelGGL((convert2d_kernel<float, float>), dim3(gp), dim3(256), 0, R.s, (float*)P, ldp, R.X32(), ldx, (int64_t)dim, r, r);
  HIP_TRY(hipGetLastError());
  return MECEFO_OK;
}

}  // extern "C"
