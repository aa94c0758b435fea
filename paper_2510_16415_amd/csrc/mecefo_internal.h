// Internal host-side interfaces between the C ABI (api.hip) and the kernel launchers.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

namespace mecefo {

enum Epilogue : int {
  EPI_STORE = 0,       // C0[row, col] = acc (activation dtype); a problem cut along K: C0 is fp32 [split][M x ldc]
  EPI_GRAD = 2,        // C0[row, col] (+)= acc                       (gradient dtype, optional accumulate)
  EPI_SWIGLU_FWD = 3,  // dual: G=C0, Z=C1, A=C2 = silu(g)*z
  EPI_SWIGLU_BWD = 4,  // dual: dA read from C0; C0=dG, C1=dZ, C2=A
  EPI_ATTN_P = 5,      // C0[row, col] = col <= row ? exp(scale * acc - rowvec[row]) : 0   (softmax from saved logsumexp)
  EPI_ATTN_DS = 6,     // C0[row, col] = C0[row, col] * (acc - rowvec[row]) * scale         (softmax backward, in place on P)
  EPI_POLY = 7,        // C0[row, col] = poly_a * (row == col) + poly_b * addend[row, col] + scale * acc; C1 (fp32) = acc
  EPI_HILO = 8,        // x = acc + addend[row, col]: C0 (fp32) = x, C1 = bf16(x), C2 = bf16(x - C1); C0 and C2 may be NULL
                       // fold_norm (bf16): x = acc / (norm of a matrix whose kNormBlocks parts have the norms in rowvec)
  EPI_RESID = 9,       // C0[row, col] = acc + C1[row, col]   (activation dtype; C1 may be C0)
  EPI_ROPE = 10,       // C0 = acc rotated: pairs (j, j + rope_half) of every head by the angle of position row % rope_seq
};

constexpr int kMaxProblems = 4;   // of one launch
constexpr int kCUs = 256;         // compute units of the chip
constexpr int kNormBlocks = 256;  // parts of a matrix whose norms are taken first

enum CausalK : int {
  CAUSAL_NONE = 0,
  CAUSAL_K_FROM_M = 1,   // terms with k < first row of the tile are zero: start the K loop there
  CAUSAL_K_UPTO_M = 2,   // terms with k > last row of the tile are zero: stop the K loop there
  CAUSAL_TILE = 3,       // output tiles entirely above the diagonal need no K loop; whole 256-blocks above it are not written
};

// One matrix product C[M x N] = sum over K-segments of opA(A_s) * opB(B_s).
//   a_kcontig: A_s is [M x K] row-major (K contiguous), else [K x M] (M contiguous).
//   b_kcontig: B_s is [N x K] row-major (K contiguous), else [K x N] (N contiguous).
// Dual products (SwiGLU epilogues) use one segment and B[0], B[1] as the gate and up
// matrices; both products share A and every size.
struct GemmProblem {
  const void* A[3];
  const void* B[3];
  void* C[3];
  int64_t lda, ldb, ldc;
  int M, N, K;
  int nseg;        // 1 to 3 K segments (ignored for dual products)
  int pad_cols;    // SwiGLU epilogues: columns [N, pad_cols) of the outputs are set to zero
  int kpad_ok;     // K-contiguous operands: bytes between K and the next multiple of 8 are known to be zero
  int splits;      // EPI_STORE: parts the contraction is cut into (0, 1: whole)
  bool whole;      // host side: never cut (the sum of the parts writes rows of ldc elements, padding included)
  bool read_parts; // host side: cut into up to kMaxNormParts parts, which the kernel behind it adds up itself
  int chunk;       // device side: K stages of a workgroup
  // Batched products (attention: one product per (sequence, head)): `batch` independent products of
  // identical size; product z = zo * batch_inner + zi reads A + zo*a_bo + zi*a_bi, etc.; all six
  // offsets are counted in operand elements (an fp32 output behind bf16 operands counts two per element).
  int batch, batch_inner;
  int64_t a_bo, a_bi, b_bo, b_bi, c_bo, c_bi;
  const float* rowvec;   // attention epilogues: fp32 per output row, product z starts at z * M
  float scale;           // attention epilogues, EPI_POLY
  const float* addend;   // EPI_POLY, EPI_HILO: fp32 [M x ldc], may be NULL (zero); may be C0 of EPI_HILO itself
  float poly_a, poly_b;  // EPI_POLY
  bool fold_norm;        // EPI_HILO: see there
  int rope_half, rope_seq;   // EPI_ROPE: half the head dimension (0: plain store) and the sequence length; rowvec and
                             // addend are the cosine and sine tables [rope_seq][rope_half]
  int causal;            // CausalK
};

// Small work of another kind that goes out in the same launch, on workgroups behind those of the products.
enum Side : int {
  SIDE_NONE = 0,
  SIDE_DGAMMA = 1,   // gain gradient from the norm backward's sums (launch_dgamma_reduce): with EPI_GRAD, both operands K-contiguous or neither
  SIDE_NORM = 2,     // norm recompute (launch_rmsnorm_fwd): with EPI_STORE, B K-strided
};
struct SideJob {
  int kind;
  int d;               // columns
  int nblk;            // SIDE_DGAMMA: rows of sums
  int out_f32, accumulate;
  float eps;           // SIDE_NORM
  int64_t rows, ld_in, ld_out;
  const void* in;      // the sums [nblk x d], or H
  const void* gamma;
  void* out;           // dgamma, or U
  float* rstd;
};

struct GemmLaunch {
  GemmProblem p[kMaxProblems];   // batch, causal and the epilogues' scalars and vectors: those of p[0] hold for all
  int nprob;
  bool a_kcontig, b_kcontig;
  int epi;          // Epilogue
  bool bf16;        // operand dtype (bf16 MFMA path) or fp32
  bool out_f32;     // EPI_GRAD: gradient buffer dtype is fp32 (else same as operands)
  int accumulate;   // EPI_GRAD
  int tile;         // EPI_ROPE: the configuration that gemm_bf16_rope_tile found for this launch
  SideJob side;
  bool side_done;   // set by the launcher: the side job is part of the launch
  uint32_t* clk;    // measurement: 64 (cycles, wall ticks) pairs written by the direct-to-LDS kernel, or NULL
};

// Records the thread-local error text returned by mecefo_last_error() and returns `status`.
int fail(int status, const char* fmt, ...) __attribute__((format(printf, 2, 3)));

// Kernels that need more than 64 KiB of dynamic LDS must have the limit raised once per device (the
// attribute belongs to the kernel's code object on that device).  One instance per kernel; ensure()
// is cheap after the first call on a device and safe from several host threads.
struct LdsLimitOnce {
  std::atomic<uint64_t> done{0};      // bit i: raised on device i (devices above 63 set it every time)
  hipError_t ensure(const void* kern, int bytes) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = dev < 64 ? (uint64_t)1 << dev : 0;
    if (bit && (done.load(std::memory_order_acquire) & bit)) return hipSuccess;
    e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e == hipSuccess && bit) done.fetch_or(bit, std::memory_order_release);
    return e;
  }
};

// Process-wide switches behind mecefo_set_option (tests and measurements; 0 = the library decides).
constexpr int kTileOptions = 11;
inline const char* const kTileOptionName[kTileOptions] = {"auto", "S", "L4", "L8R", "L8", "S4", "T", "T2", "K", "LT", "X"};
struct Options {
  std::atomic<int> tile{0};        // bf16 GEMM configuration, index into kTileOptionName
  std::atomic<int> attn_gemm{0};   // 1: attention through batched GEMM launches instead of the fused kernels
};
Options& options();

// Raise the dynamic-LDS limit of every kernel that needs it on the current device (what the first
// launch of each kernel would otherwise do): mecefo_init.
hipError_t prepare_gemm_bf16_nt();
hipError_t prepare_gemm_bf16_nn();
hipError_t prepare_gemm_bf16_tn();
hipError_t prepare_gemm_f32();
// The configuration with which the bf16 launch (NT layout) carries EPI_ROPE for heads of dimension dh; -1: none.
int gemm_bf16_rope_tile(const GemmLaunch& g, int dh);
// The tile on which dA = dY Wd and the recompute whose epilogue reads it (one bf16 product each) go out as one launch, -1
// where two are shorter.  cost: us that the one launch costs besides.
int gemm_bf16_pair_tile(const GemmLaunch& dA, const GemmLaunch& rec, float cost);
hipError_t launch_gemm_bf16_pair(const GemmLaunch& dA, const GemmLaunch& rec, int tile, hipStream_t s);
hipError_t prepare_attention_fwd();
hipError_t prepare_attention_bwd();

// Returns hipSuccess or the launch error.  Only enqueues.
hipError_t launch_gemm(GemmLaunch& g, hipStream_t stream);
hipError_t launch_gemm_bf16(GemmLaunch& g, hipStream_t stream);
hipError_t launch_gemm_f32(GemmLaunch& g, hipStream_t stream);
void f32_plan_splits(GemmLaunch& g, int most);   // cuts every problem of the launch into the same number of parts
void f32_plan_parts(GemmLaunch& g, int64_t room);   // cuts the problem with read_parts, into `room` fp32 elements at most
bool f32_far(const GemmLaunch& g);

// Elementwise / reduction kernels (elementwise.hip).  `bf16` selects the storage type.
// cos / sin of position * theta^(-2j/dh) for every position < seq and j < half = dh / 2.
struct RopeTables { float* cs; float* sn; int seq, half; double theta; };
inline unsigned rope_table_blocks(const RopeTables& t) { return (unsigned)((t.seq * t.half + 255) / 256); }

// `tables`: written by workgroups of their own in the same launch, or NULL (a launch of 5 us less; the forward of 4096 tokens,
// d 1024: 157.5 -> 154.7 us).
hipError_t launch_rmsnorm_fwd(bool bf16, const void* H, int64_t ldh, const void* gamma, float eps,
                              void* U, int64_t ldu, float* rstd, int64_t b, int d, hipStream_t s,
                              const RopeTables* tables = nullptr);
// dX = dOut + rmsnorm_backward(dU); sums of the gain gradient over groups of rows go to dg_partial [nblk x d], of which
// the launch says how many there are (rmsnorm_bwd_blocks, or more where dg_room, in floats, has space for them).  dU: in
// the storage type (parts 0), or the sum of `parts` fp32 products [b x lddu], part_stride elements apart
// (rmsnorm_bwd_takes_parts).
struct NormBwd {
  const void* dU; int64_t lddu; int parts; int64_t part_stride;
  const void* H; int64_t ldh;
  const float* rstd; const void* gamma;
  const void* dOut; int64_t lddo;
  void* dX; int64_t lddx;
  float* dg_partial; int64_t dg_room;
  int64_t b; int d;
};
constexpr int kMaxNormParts = 4;
inline bool rmsnorm_bwd_parts_width(bool bf16, int d) { return d <= 2048 && d % (bf16 ? 8 : 4) == 0; }   // what is built
bool rmsnorm_bwd_takes_parts(bool bf16, const NormBwd& n);
hipError_t launch_rmsnorm_bwd(bool bf16, const NormBwd& n, int* nblk, hipStream_t s);
int rmsnorm_bwd_blocks(int64_t b);
hipError_t launch_dgamma_reduce(const float* dg_partial, int nblk, int d, void* dgamma, bool out_f32,
                                bool bf16, int accumulate, hipStream_t s);
// dX = dOut + dU  (no-norm variant)
hipError_t launch_add(bool bf16, const void* a, int64_t lda, const void* bsrc, int64_t ldb, void* out,
                      int64_t ldo, int64_t rows, int cols, hipStream_t s);
// out[0 .. n) (activation dtype, 16-byte aligned) = sum over the parts of part[k][0 .. n), for up to kMaxProblems jobs
struct SumJob { const float* part; void* out; int64_t n; int parts; };
hipError_t launch_sum_parts(bool bf16, const SumJob* jobs, int n, hipStream_t s);
// Standalone SwiGLU backward from saved G, Z: reads dA (in DG), writes DG=dG, DZ=dZ, AA=A; pads zeroed.
hipError_t launch_swiglu_bwd(bool bf16, const void* G, const void* Z, int64_t ldgz, void* DG, void* DZ,
                             void* AA, int64_t ldf, int64_t b, int f, int pad_cols, hipStream_t s);


// Attention helpers (attention.hip).
// In-place rotary rotation of two token-major [tokens x heads*dh] tensors (inverse: the transpose, for gradients).
hipError_t launch_rope(bool bf16, void* X0, void* X1, int64_t ldx, const float* cs, const float* sn, int64_t tokens,
                       int seq, int heads, int dh, bool inverse, hipStream_t s);
// Causal row softmax of `nprod` fp32 score matrices [seq x lds]: P (storage type) and the log-sum-exp L.
hipError_t launch_softmax_rows(bool bf16, const float* S, int64_t lds, void* P, int64_t ldp, float* L, int nprod,
                               int seq, float scale, hipStream_t s);
// D[(sequence*heads + head)*seq + s] = sum over the head's columns of dO * O.
hipError_t launch_attn_rowdot(bool bf16, const void* dO, int64_t lddo, const void* O, int64_t ldo, float* D,
                              int64_t tokens, int seq, int heads, int dh, hipStream_t s);


// Fused causal attention backward for dK, dV (attention_bwd.hip): also writes dS = P (dP - D) scale
// (bf16, [batch*heads][seq x ldp], zeros above the diagonal inside the diagonal 256-blocks) for the
// batched dQ = dS K product that follows.  bf16, head dimension 64 or 128.
bool attn_bwd_fused_supported(bool bf16, int dh, int seq, int64_t ldp);
hipError_t launch_attn_bwd_kv(const void* Q, const void* K, const void* V, int64_t ld_in, const void* dO,
                              void* dK, void* dV, int64_t ld_ws, const float* L, const float* D, void* dS,
                              int64_t ldp, int batch, int seq, int heads, int dh, float scale, hipStream_t s);


// Fused causal attention forward: O = softmax(scale Q K^T) V and the row log-sum-exp L [batch*heads][seq],
// no score or probability buffer.  Q, K, V, O token-major with row stride ld (elements), head h at
// columns h*dh.  bf16, head dimension 64 or 128, ld a multiple of 8.
bool attn_fwd_fused_supported(bool bf16, int dh, int seq, int64_t ld);
hipError_t launch_attn_fwd(const void* Q, const void* K, const void* V, void* O, int64_t ld, float* L, int batch,
                           int seq, int heads, int dh, float scale, hipStream_t s);

}  // namespace mecefo
