// C ABI of the degraded block backward: argument validation, workspace carving and the
// order in which the kernels are enqueued.  Every arithmetic step runs in the kernels.
#include <stdarg.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <vector>

#include "../../include/mecefo.h"
#include "gemm_bf16_launch.hip.h"
#include "mecefo_internal.h"

using namespace mecefo;

namespace mecefo {
hipError_t launch_gemm(GemmLaunch& g, hipStream_t s) {
  if (!g.bf16) return launch_gemm_f32(g, s);
  if (g.a_kcontig && g.b_kcontig) return launch_gemm_bf16_nt(g, s);
  if (g.a_kcontig && !g.b_kcontig) return launch_gemm_bf16_nn(g, s);
  if (!g.a_kcontig && !g.b_kcontig) return launch_gemm_bf16_tn(g, s);
  return hipErrorInvalidValue;
}
}  // namespace mecefo

namespace mecefo {
Options& options() {
  static Options o;
  return o;
}

thread_local char g_err[512] = "";

int fail(int st, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
  return st;
}
}  // namespace mecefo

namespace {

// Status-typed front of mecefo::fail; a macro so that the compiler still checks the format string
// against the arguments at every call site.
#define fail(st, ...) ((mecefo_status_t)mecefo::fail((int)(st), __VA_ARGS__))

constexpr int64_t kMaxBytes = (int64_t)1 << 31;

inline int64_t up(int64_t x, int64_t a) { return (x + a - 1) / a * a; }

struct Ctx {
  const mecefo_ffn_desc_t* d;
  bool bf16;
  int esz;          // bytes per activation element
  int64_t b;
  int dm, ff;
  int64_t ldf;      // row stride of internal [b x f] buffers
  bool grad_f32;
};

mecefo_status_t check_desc(const mecefo_ffn_desc_t* d, Ctx* c) {
  if (!d) return fail(MECEFO_ERR_INVALID_ARG, "descriptor is NULL");
  if (d->dtype != MECEFO_F32 && d->dtype != MECEFO_BF16)
    return fail(MECEFO_ERR_INVALID_ARG, "dtype must be MECEFO_F32 or MECEFO_BF16");
  if (d->grad_dtype != MECEFO_F32 && d->grad_dtype != d->dtype)
    return fail(MECEFO_ERR_UNSUPPORTED, "grad_dtype must be MECEFO_F32 or equal to dtype");
  if (d->tokens < 0 || d->d_model < 1 || d->d_ff < 1)
    return fail(MECEFO_ERR_INVALID_ARG, "tokens >= 0, d_model >= 1, d_ff >= 1 required");
  if (d->ld_act_d < d->d_model || d->ld_act_f < d->d_ff || d->ld_w_fd < d->d_model || d->ld_w_df < d->d_ff)
    return fail(MECEFO_ERR_INVALID_ARG, "a row stride is smaller than the logical width");
  c->d = d;
  c->bf16 = d->dtype == MECEFO_BF16;
  c->esz = c->bf16 ? 2 : 4;
  c->b = d->tokens;
  c->dm = d->d_model;
  c->ff = d->d_ff;
  c->ldf = up(d->d_ff, 8);
  c->grad_f32 = d->grad_dtype == MECEFO_F32;
  if (c->bf16) {
    if (d->d_model % 8)
      return fail(MECEFO_ERR_UNSUPPORTED, "bf16 path needs d_model to be a multiple of 8 (got %d)", d->d_model);
    if (d->ld_act_d % 8 || d->ld_act_f % 8 || d->ld_w_fd % 8 || d->ld_w_df % 8)
      return fail(MECEFO_ERR_INVALID_ARG,
                  "bf16 path needs every row stride to be a multiple of 8 elements (pad d_ff=%d to %lld)",
                  d->d_ff, (long long)up(d->d_ff, 8));
  }
  const int64_t big = d->tokens * (d->ld_act_f > d->ld_act_d ? d->ld_act_f : d->ld_act_d);
  const int64_t wbig = (int64_t)d->d_ff * d->ld_w_fd > (int64_t)d->d_model * d->ld_w_df
                           ? (int64_t)d->d_ff * d->ld_w_fd : (int64_t)d->d_model * d->ld_w_df;
  if (big * c->esz >= kMaxBytes || wbig * 4 >= kMaxBytes)
    return fail(MECEFO_ERR_UNSUPPORTED, "a tensor reaches 2 GiB; split the token batch");
  return MECEFO_OK;
}

mecefo_status_t check_ptr(const Ctx& c, const void* p, const char* name, bool required = true) {
  if (!p) return required ? fail(MECEFO_ERR_INVALID_ARG, "%s is NULL", name) : MECEFO_OK;
  if (((uintptr_t)p) % (c.bf16 ? 16 : 4)) return fail(MECEFO_ERR_INVALID_ARG, "%s is not %d-byte aligned", name, c.bf16 ? 16 : 4);
  return MECEFO_OK;
}

// Bytes spanned by a [b x d_model] activation tensor with row stride ld.
size_t act_span(const Ctx& c, int64_t ld) { return c.b > 0 ? (size_t)(((c.b - 1) * ld + c.dm) * c.esz) : 0; }

// An output may coincide with an input it is allowed to overwrite (same pointer), or lie apart from it;
// a partial overlap would let the kernels read rows that are already overwritten.
mecefo_status_t check_alias(const void* out, const char* out_name, const void* in, const char* in_name, size_t bytes) {
  if (!out || !in || out == in || bytes == 0) return MECEFO_OK;
  const uintptr_t a = (uintptr_t)out, b = (uintptr_t)in;
  if (a < b + bytes && b < a + bytes)
    return fail(MECEFO_ERR_INVALID_ARG, "%s overlaps %s without being equal to it", out_name, in_name);
  return MECEFO_OK;
}

mecefo_status_t check_proj(const Ctx& c, const mecefo_proj_t& P, int dim, const char* name) {
  if (!P.P) return fail(MECEFO_ERR_INVALID_ARG, "projection %s is NULL", name);
  if (P.r < 1 || P.r > dim) return fail(MECEFO_ERR_INVALID_ARG, "projection %s: rank %d outside [1, %d]", name, P.r, dim);
  if (P.ld < P.r) return fail(MECEFO_ERR_INVALID_ARG, "projection %s: ld %lld < r %d", name, (long long)P.ld, P.r);
  if (c.bf16 && (P.ld % 8 || ((uintptr_t)P.P) % 16))
    return fail(MECEFO_ERR_INVALID_ARG, "projection %s: bf16 path needs ld %% 8 == 0 and a 16-byte aligned pointer", name);
  // the bf16 kernels address a whole operand with 32-bit offsets: rows behind 2 GiB would read as zeros
  if (c.bf16 && dim > 1 && P.ld > (0x7FFFFFFF / 2 - P.r) / (dim - 1))
    return fail(MECEFO_ERR_UNSUPPORTED, "projection %s: %d rows of stride %lld reach 2 GiB", name, dim, (long long)P.ld);
  return MECEFO_OK;
}

#define TRY(x) do { mecefo_status_t st__ = (x); if (st__ != MECEFO_OK) return st__; } while (0)
#define HIP_TRY(x) do { hipError_t e__ = (x); if (e__ != hipSuccess) return fail(MECEFO_ERR_LAUNCH, "%s: %s", #x, hipGetErrorString(e__)); } while (0)

// ---- optional per-stage timing (measurement only) --------------------------------------
constexpr int kClkPairs = 64;      // (cycles, wall ticks) pairs per stage launch
struct Profiler {
  bool on = false;
  std::vector<hipEvent_t> ev;     // pairs (start, stop)
  std::vector<int> stage;
  size_t used = 0;                // events used
  uint32_t* clk = nullptr;        // device: [stage launches][kClkPairs][2], zero-filled by mecefo_profile_enable
  uint32_t* cur_clk = nullptr;    // slot of the stage that is being enqueued
  double mhz[MECEFO_STAGE_COUNT] = {};
} g_prof;

struct StageTimer {
  hipStream_t s;
  size_t at = 0;      // first event of the pair, this stage's from here on
  bool active;
  StageTimer(int stage, hipStream_t stream) : s(stream), active(false) {
    if (g_prof.on && g_prof.used + 2 <= g_prof.ev.size()) {
      active = true;
      at = g_prof.used;
      g_prof.used += 2;
      g_prof.stage[at / 2] = stage;
      g_prof.cur_clk = g_prof.clk ? g_prof.clk + (at / 2) * kClkPairs * 2 : nullptr;
      (void)hipEventRecord(g_prof.ev[at], s);
    }
  }
  ~StageTimer() {
    if (active) {
      (void)hipEventRecord(g_prof.ev[at + 1], s);
      g_prof.cur_clk = nullptr;
    }
  }
};
#define STAGE(id, stream) StageTimer stage_timer__((id), (stream))

// ---- workspace ------------------------------------------------------------------------
struct Workspace {
  // offsets in bytes from the (256-byte aligned) workspace base
  size_t U, rstd, DG, DZ, AA, dU, T[3], C[3], partial, dgp, parts, total;
  int64_t room, parts_room;      // fp32 elements of the partial buffer, and of the one that keeps the parts of dU
  int splits;
  int64_t c_elems[3];
};

// Most parts the token contraction of Eq. (2) may be cut into (what the workspace holds partials for): the outputs
// ([f x r], [d x r]) are small, so the long token dimension gives workgroups for 256 CUs.  The launch takes as many of
// them as its cost model finds worth their summation.
int choose_splits(const Ctx& c, const int64_t c_rows[3], const int r[3]) {
  int tiles_l = 0, tiles_s = 0, tiles_f = 0;
  for (int i = 0; i < 3; ++i) {
    if (r[i] <= 0) continue;
    tiles_l += cdiv((int)c_rows[i], 256) * cdiv(r[i], 256);
    tiles_s += cdiv((int)c_rows[i], 128) * cdiv(r[i], 128);
    tiles_f += cdiv((int)c_rows[i], 64) * cdiv(r[i], 64);
  }
  int tiles, ktiles, target;
  if (!c.bf16) { tiles = tiles_f; ktiles = cdiv((int)c.b, 16); target = 512; }
  else if (tiles_l >= 160) { tiles = tiles_l; ktiles = cdiv((int)c.b, 64); target = 256; }
  else {
    // Mid-size layers: 256 x 256 tiles cut along the tokens into just enough parts for half the chip, as long
    // as every part keeps eight K stages.
    ktiles = cdiv((int)c.b, 64);
    const int s_l = tiles_l > 0 ? cdiv(128, tiles_l) : 0;
    if (s_l >= 1 && s_l <= 16 && ktiles / s_l >= 8) return s_l;
    tiles = tiles_s; target = 512;
  }
  if (tiles == 0) return 1;
  int s = cdiv(target, tiles);
  const int smax = ktiles / 4 > 1 ? ktiles / 4 : 1;
  if (s > smax) s = smax;
  if (s > 16) s = 16;
  return s < 1 ? 1 : s;
}

// Most K splits of a launch that stores activation-dtype outputs but has too few 256 x 256 tiles to fill
// the chip (mid-size layers: dU = dG Wg + dZ Wu with a small d, the projections with a small r): the long
// contraction may be cut until about 256 workgroups exist, fp32 partials are summed in order.
constexpr int kMaxStoreSplits = 4;
int store_splits(bool bf16, int tiles_large, int min_stages) {
  if (!bf16 || tiles_large <= 0 || tiles_large >= 128 || min_stages < 32) return 1;
  int sp = cdiv(256, tiles_large);
  if (sp > min_stages / 8) sp = min_stages / 8;
  if (sp > kMaxStoreSplits) sp = kMaxStoreSplits;
  return sp < 1 ? 1 : sp;
}
int store_splits_du(const Ctx& c) {   // dU [b x d], two K segments of length f
  return store_splits(c.bf16, cdiv((int)c.b, 256) * cdiv(c.dm, 256), 2 * cdiv(c.ff, 64));
}
int store_splits_project(const Ctx& c, const int r[3], mecefo_side_t side) {   // T_i [b x r_i]
  int tiles = 0, stages = 0;
  for (int i = 0; i < 3; ++i) {
    if (r[i] <= 0) continue;
    tiles += cdiv((int)c.b, 256) * cdiv(r[i], 256);
    const int k = side == MECEFO_SIDE_INPUT ? (i < 2 ? c.dm : c.ff) : (i < 2 ? c.ff : c.dm);
    if (cdiv(k, 64) > stages) stages = cdiv(k, 64);      // the longest contraction sets the pace of the launch
  }
  if (tiles <= 0 || !c.bf16 || tiles >= 128 || stages < 16) return 1;
  // as many parts as fit the chip in one go, none shorter than four K stages of the longest problem
  int sp = 256 / tiles;
  if (sp > stages / 4) sp = stages / 4;
  if (sp > 8) sp = 8;
  return sp < 1 ? 1 : sp;
}

// Parts of dU that the norm backward adds up: where there are any they outlive the token contraction, which has the
// partial buffer, so they have a buffer of their own.  Workspaces sized without it are taken too (with_parts = false).
int kept_parts(const Ctx& c) {
  if (!rmsnorm_bwd_parts_width(c.bf16, c.dm)) return 0;
  if (c.bf16) return store_splits_du(c) > 1 ? kMaxNormParts : 0;
  return (c.b + 31) / 32 * ((c.dm + 31) / 32) <= kCUs / 2 ? kMaxNormParts : 0;
}

Workspace layout(const Ctx& c, const int r[3], mecefo_side_t side, int force_splits, bool with_parts) {
  Workspace w;
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off += (size_t)up((int64_t)bytes, 256); return o; };
  const size_t act_d = (size_t)c.b * c.dm * c.esz, act_f = (size_t)c.b * c.ldf * c.esz;
  w.U = take(act_d);
  w.rstd = take((size_t)c.b * 4);
  w.DG = take(act_f);
  w.DZ = take(act_f);
  w.AA = take(act_f);
  w.dU = take(act_d);
  // C_i rows: SIDE_INPUT: gate/up -> f, down -> d (output dim); SIDE_OUTPUT: gate/up -> d, down -> f.
  int64_t c_rows[3];
  c_rows[0] = c_rows[1] = side == MECEFO_SIDE_INPUT ? c.ff : c.dm;
  c_rows[2] = side == MECEFO_SIDE_INPUT ? c.dm : c.ff;
  int64_t sum_c = 0;
  for (int i = 0; i < 3; ++i) {
    const int64_t rr = up(r[i] > 0 ? r[i] : 0, 8);
    w.T[i] = take((size_t)c.b * rr * c.esz);
    w.c_elems[i] = c_rows[i] * rr;
    w.C[i] = take((size_t)w.c_elems[i] * c.esz);
    sum_c += c_rows[i] * rr;
  }
  w.splits = force_splits > 0 ? force_splits : choose_splits(c, c_rows, r);
  // one partial buffer serves the launches that split K, one after the other on the stream
  size_t partial = w.splits > 1 ? (size_t)w.splits * sum_c * 4 : 0;
  const int sdu = store_splits_du(c), spr = store_splits_project(c, r, side);
  if (sdu > 1 && (size_t)sdu * c.b * c.dm * 4 > partial) partial = (size_t)sdu * c.b * c.dm * 4;
  if (spr > 1) {
    size_t t = 0;
    for (int i = 0; i < 3; ++i) t += (size_t)c.b * up(r[i] > 0 ? r[i] : 0, 8) * 4;
    if ((size_t)spr * t > partial) partial = (size_t)spr * t;
  }
  w.partial = take(partial);
  w.room = (int64_t)(partial / 4);
  w.dgp = take((size_t)rmsnorm_bwd_blocks(c.b) * c.dm * 4);
  w.parts_room = with_parts ? kept_parts(c) * c.b * c.dm : 0;
  w.parts = take((size_t)w.parts_room * 4);
  w.total = off + 256;   // slack for aligning the caller's base pointer
  return w;
}

struct Bufs { char* base; Workspace w; };

mecefo_status_t carve(const Ctx& c, const int r[3], mecefo_side_t side, void* ws, size_t ws_bytes, Bufs* out) {
  Workspace w = layout(c, r, side, 0, true);
  if (w.total > ws_bytes) w = layout(c, r, side, 0, false);
  while (w.total > ws_bytes && w.splits > 1) w = layout(c, r, side, w.splits - 1, false);
  if (w.total > ws_bytes)
    return fail(MECEFO_ERR_WORKSPACE_TOO_SMALL, "workspace has %zu bytes, %zu needed", ws_bytes, w.total);
  if (!ws) return fail(MECEFO_ERR_INVALID_ARG, "workspace is NULL");
  out->base = (char*)up((int64_t)(uintptr_t)ws, 256);
  out->w = w;
  return MECEFO_OK;
}

GemmLaunch new_launch(const Ctx& c, bool akc, bool bkc, int epi) {
  GemmLaunch g;
  memset(&g, 0, sizeof(g));
  g.a_kcontig = akc;
  g.b_kcontig = bkc;
  g.epi = epi;
  g.bf16 = c.bf16;
  g.out_f32 = c.grad_f32;
  g.clk = g_prof.cur_clk;
  return g;
}

GemmProblem prob(const void* A0, const void* A1, int64_t lda, const void* B0, const void* B1, int64_t ldb,
                 void* C0, void* C1, void* C2, int64_t ldc, int M, int N, int K, int nseg, int pad_cols = 0) {
  GemmProblem p;
  memset(&p, 0, sizeof(p));
  p.A[0] = A0; p.A[1] = A1 ? A1 : A0;
  p.B[0] = B0; p.B[1] = B1 ? B1 : B0;
  p.C[0] = C0; p.C[1] = C1; p.C[2] = C2;
  p.lda = lda; p.ldb = ldb; p.ldc = ldc;
  p.M = M; p.N = N; p.K = K; p.nseg = nseg; p.pad_cols = pad_cols;
  return p;
}

// A store launch into the library's own buffers, its problems cut along K as their `splits` say (bf16_plan_splits):
// those write fp32 parts into `partial`, one problem's behind the other's, which one more launch sums.
// A problem with read_parts writes them into `parts`, and `kept` says how many there are.
struct Parts { const float* p = nullptr; int n = 0; };
mecefo_status_t launch_store(const Ctx& c, const Bufs& bf, GemmLaunch& g, hipStream_t s, Parts* kept = nullptr) {
  SumJob jobs[kMaxProblems];
  int n = 0;
  float* partial = (float*)(bf.base + bf.w.partial);
  for (int i = 0; i < g.nprob; ++i) {
    GemmProblem& p = g.p[i];
    if (p.splits <= 1) continue;
    if (p.read_parts) {
      p.C[0] = bf.base + bf.w.parts;
      *kept = Parts{(const float*)p.C[0], p.splits};
      continue;
    }
    jobs[n++] = SumJob{partial, p.C[0], (int64_t)p.M * p.ldc, p.splits};
    p.C[0] = partial;
    partial += (int64_t)p.splits * p.M * p.ldc;
  }
  HIP_TRY(launch_gemm(g, s));
  if (n > 0) HIP_TRY(launch_sum_parts(c.bf16, jobs, n, s));
  return MECEFO_OK;
}

// ---- norm recompute ----
SideJob norm_job(const Ctx& c, const void* H, int64_t ldh, const void* gamma, void* U, float* rstd) {
  SideJob j = {SIDE_NORM, c.dm, 0, 0, 0, c.d->rms_eps, c.b, ldh, c.dm, H, gamma, U, rstd};
  return j;
}
mecefo_status_t norm_forward(const Ctx& c, const SideJob& j, hipStream_t s) {
  STAGE(MECEFO_STAGE_NORM_FWD, s);
  HIP_TRY(launch_rmsnorm_fwd(c.bf16, j.in, j.ld_in, j.gamma, j.eps, j.out, j.ld_out, j.rstd, j.rows, j.d, s));
  return MECEFO_OK;
}
// dA does not read U: the norm recompute of a small layer rides on its launch (a launch less, 3.5 us).  Larger ones keep
// their own, with more waves in flight than the LDS of the product leaves room for.
bool norm_rides(const Ctx& c) { return c.b * c.dm * c.esz <= (int64_t)4 << 20; }

// dA = dY Wd  ->  recompute G, Z from U and apply the SwiGLU backward in the epilogue
// (DG = dG, DZ = dZ, AA = A).   Sec. 3.3 (Rcomp).
mecefo_status_t recompute(const Ctx& c, const Bufs& bf, const void* U, int64_t ldu, const void* dY,
                                    int64_t lddy, const void* Wg, const void* Wu, const void* Wd,
                                    const void* Gsaved, const void* Zsaved, hipStream_t s, const SideJob* norm = nullptr) {
  const mecefo_ffn_desc_t& d = *c.d;
  char* base = bf.base;
  void* DG = base + bf.w.DG; void* DZ = base + bf.w.DZ; void* AA = base + bf.w.AA;
  const int b = (int)c.b;
  if (b == 0) return MECEFO_OK;
  GemmLaunch down = new_launch(c, true, false, EPI_STORE);      // dA = dY Wd   [b x f], K = d
  down.nprob = 1;
  down.p[0] = prob(dY, nullptr, lddy, Wd, nullptr, d.ld_w_df, DG, nullptr, nullptr, c.ldf, b, c.ff, c.dm, 1);
  GemmLaunch rec = new_launch(c, true, true, EPI_SWIGLU_BWD);   // G = U Wg^T, Z = U Wu^T, the SwiGLU backward in the epilogue
  rec.nprob = 1;
  rec.p[0] = prob(U, nullptr, ldu, Wg, Wu, d.ld_w_fd, DG, DZ, AA, c.ldf, b, c.ff, c.dm, 1, (int)c.ldf);
  // a norm recompute that would ride on dA is a launch of its own then
  const int pair = c.bf16 && !Gsaved ? gemm_bf16_pair_tile(down, rec, norm ? 3.2f : 0.f) : -1;
  if (pair >= 0) {
    if (norm) TRY(norm_forward(c, *norm, s));
    STAGE(MECEFO_STAGE_RECOMPUTE, s);
    rec.clk = nullptr;
    HIP_TRY(launch_gemm_bf16_pair(down, rec, pair, s));
    return MECEFO_OK;
  }
  {
    STAGE(MECEFO_STAGE_DGRAD_DOWN, s);
    down.clk = g_prof.cur_clk;
    if (norm) down.side = *norm;
    HIP_TRY(launch_gemm(down, s));
  }
  if (norm && !down.side_done) TRY(norm_forward(c, *norm, s));
  if (Gsaved) {
    STAGE(MECEFO_STAGE_SWIGLU_BWD, s);
    HIP_TRY(launch_swiglu_bwd(c.bf16, Gsaved, Zsaved, d.ld_act_f, DG, DZ, AA, c.ldf, c.b, c.ff, (int)c.ldf, s));
  } else {
    STAGE(MECEFO_STAGE_RECOMPUTE, s);
    rec.clk = g_prof.cur_clk;
    HIP_TRY(launch_gemm(rec, s));
  }
  return MECEFO_OK;
}

// dU = dG Wg + dZ Wu   [b x d], two K segments of length f
GemmProblem dgrad_problem(const Ctx& c, const Bufs& bf, const void* Wg, const void* Wu, void* dU, int64_t lddu) {
  GemmProblem p = prob(bf.base + bf.w.DG, bf.base + bf.w.DZ, c.ldf, Wg, Wu, c.d->ld_w_fd, dU, nullptr, nullptr, lddu,
                       (int)c.b, c.dm, c.ff, 2);
  p.kpad_ok = 1;   // DG / DZ padding columns were written as zeros; the weight rows are predicated exactly
  p.whole = dU != bf.base + bf.w.dU;
  return p;
}
// kept: not NULL where the norm backward behind it takes the parts of dU (norm_bwd_reads_parts).
mecefo_status_t dgrad(const Ctx& c, const Bufs& bf, const void* Wg, const void* Wu, void* dU, int64_t lddu, hipStream_t s,
                      Parts* kept = nullptr) {
  if (!dU || c.b == 0) return MECEFO_OK;
  STAGE(MECEFO_STAGE_DGRAD_GATE_UP, s);
  GemmLaunch g = new_launch(c, true, false, EPI_STORE);
  g.nprob = 1;
  g.p[0] = dgrad_problem(c, bf, Wg, Wu, dU, lddu);
  g.p[0].read_parts = kept != nullptr;
  if (c.bf16) bf16_plan_splits(g, bf.w.room, bf.w.parts_room);
  else if (kept) f32_plan_parts(g, bf.w.parts_room);
  return launch_store(c, bf, g, s, kept);
}

// ---- norm backward ----
// dX = dOut + normbwd(dU) and the gain gradient.  dU is the workspace's own [b x d] buffer, or parts of it, and then that
// buffer takes the sums of the gain gradient.
NormBwd norm_bwd_args(const Ctx& c, const Bufs& bf, const Workspace& w, const Parts& parts, const void* H, int64_t ldh,
                      const void* gamma, const void* dOut, int64_t lddo, void* dX, int64_t lddx, bool want_dgamma) {
  char* base = bf.base;
  NormBwd n = {base + w.dU, c.dm, 0, 0, H, ldh, (const float*)(base + w.rstd), gamma, dOut, lddo, dX, lddx,
               (float*)(base + w.dgp), (int64_t)rmsnorm_bwd_blocks(c.b) * c.dm, c.b, c.dm};
  if (parts.n > 1) {
    n.dU = parts.p; n.parts = parts.n; n.part_stride = c.b * c.dm;
    if ((c.b + 3) / 4 * c.dm <= c.b * c.dm * c.esz / 4) {
      n.dg_partial = (float*)(base + w.dU);
      n.dg_room = c.b * c.dm * c.esz / 4;
    }
  }
  if (!want_dgamma) n.dg_partial = nullptr;
  return n;
}
// `later`: receives the sum of the gain gradient as a side job for a launch behind this one, else it is launched here.
mecefo_status_t norm_backward(const Ctx& c, const NormBwd& n, void* dgamma, int accumulate, hipStream_t s, SideJob* later = nullptr) {
  STAGE(MECEFO_STAGE_NORM_BWD, s);
  int nblk = 0;
  if (c.b > 0) HIP_TRY(launch_rmsnorm_bwd(c.bf16, n, &nblk, s));
  if (!dgamma) return MECEFO_OK;
  if (later) *later = SideJob{SIDE_DGAMMA, c.dm, nblk, c.grad_f32, accumulate, 0.f, 0, 0, 0, n.dg_partial, nullptr, dgamma, nullptr};
  else HIP_TRY(launch_dgamma_reduce(n.dg_partial, nblk, c.dm, dgamma, c.grad_f32, c.bf16, accumulate, s));
  return MECEFO_OK;
}
// The sum of the gain gradient, where the launch that was to carry it as its side job did not.
mecefo_status_t dgamma_left(const Ctx& c, const GemmLaunch& g, hipStream_t s) {
  const SideJob& j = g.side;
  if (j.kind != SIDE_DGAMMA || g.side_done) return MECEFO_OK;
  STAGE(MECEFO_STAGE_NORM_BWD, s);
  HIP_TRY(launch_dgamma_reduce((const float*)j.in, j.nblk, j.d, j.out, j.out_f32, c.bf16, j.accumulate, s));
  return MECEFO_OK;
}
// Whether these arguments suit the kernel that adds up parts, and the workspace keeps them.
bool norm_bwd_reads_parts(const Ctx& c, const Bufs& bf, NormBwd n) {
  if (bf.w.parts_room == 0) return false;
  n.dU = bf.base + bf.w.parts;
  n.parts = 2;
  n.part_stride = c.b * c.dm;
  return rmsnorm_bwd_takes_parts(c.bf16, n);
}

// The three products of Eq. (2) for the FFN matrices that take it, T = X P, C = Gy^T T, dW = C P^T (SIDE_INPUT) or
// T = Gy P, C = X^T T, dW = P C^T (SIDE_OUTPUT), with (Gy, X) = (dG, U) for gate, (dZ, U) for up, (dY, A) for down.
struct LowRank {
  const void* Gy[3]; const void* X[3];
  int64_t ldgy[3], ldx[3], ldt[3], lddw[3];
  int m_out[3], n_in[3];      // rows and columns of dW
  void* T[3]; void* C[3];
  const mecefo_proj_t* P;
  bool in;                    // SIDE_INPUT
  int lr[3], ex[3], n_lr, n_ex;      // matrices that take Eq. (2), and those that take the exact weight gradient
};
LowRank low_rank(const Ctx& c, const Bufs& bf, const void* U, int64_t ldu, const void* dY, int64_t lddy,
                 const mecefo_proj_t P[3], mecefo_side_t side, int exact_mask) {
  const mecefo_ffn_desc_t& d = *c.d;
  char* base = bf.base;
  LowRank q = {{base + bf.w.DG, base + bf.w.DZ, dY}, {U, U, base + bf.w.AA}, {c.ldf, c.ldf, lddy}, {ldu, ldu, c.ldf}, {},
               {d.ld_w_fd, d.ld_w_fd, d.ld_w_df}, {c.ff, c.ff, c.dm}, {c.dm, c.dm, c.ff}, {}, {}, P,
               side == MECEFO_SIDE_INPUT, {}, {}, 0, 0};
  for (int i = 0; i < 3; ++i) {
    q.ldt[i] = up(P[i].r, 8); q.T[i] = base + bf.w.T[i]; q.C[i] = base + bf.w.C[i];
    if (exact_mask & (1 << i)) q.ex[q.n_ex++] = i;
    else q.lr[q.n_lr++] = i;
  }
  return q;
}
// T of matrix i: contraction over the projected dimension
GemmProblem project_problem(const Ctx& c, const Bufs& bf, const LowRank& q, int i) {
  const void* a_op = q.in ? q.X[i] : q.Gy[i];
  GemmProblem p = prob(a_op, nullptr, q.in ? q.ldx[i] : q.ldgy[i], q.P[i].P, nullptr, q.P[i].ld, q.T[i], nullptr, nullptr,
                       q.ldt[i], (int)c.b, q.P[i].r, q.in ? q.n_in[i] : q.m_out[i], 1);
  // the K-contiguous operand is one of the library's own zero-padded [b x f] buffers (A, dG, dZ)
  p.kpad_ok = (a_op == bf.base + bf.w.AA || a_op == bf.base + bf.w.DG || a_op == bf.base + bf.w.DZ) ? 1 : 0;
  return p;
}

// dU and the projections of Eq. (2), in one launch where that is shorter than two.  Both are few long products: dU
// [b x d] walks 2 f, the down projection's T [b x r] walks f (SIDE_INPUT) on a fraction of the chip, the others d.
mecefo_status_t dgrad_and_project(const Ctx& c, const Bufs& bf, const LowRank& q, const void* Wg, const void* Wu,
                                  void* dU, int64_t lddu, hipStream_t s, Parts* kept = nullptr) {
  if (c.b == 0) return MECEFO_OK;
  GemmLaunch project = new_launch(c, true, false, EPI_STORE);
  for (int j = 0; j < q.n_lr; ++j) project.p[project.nprob++] = project_problem(c, bf, q, q.lr[j]);
  if (dU && q.n_lr > 0) {
    GemmLaunch both = project, alone = project;
    alone.p[0] = dgrad_problem(c, bf, Wg, Wu, dU, lddu);
    alone.p[0].read_parts = kept != nullptr;
    both.p[both.nprob++] = alone.p[0];
    alone.nprob = 1;
    // large layers, where the two launches fill the chip by themselves, keep them (1456 us against 1474 for 8192 tokens,
    // d 4096, f 11008).  fp32 always merges: calls with two launches / one, us, [256 x 256], f 688: 42.6 / 36.8;
    // [1024 x 512], f 1376: 190 / 188; [4096 x 512], f 1376: 488 / 475; [4096 x 1024], f 2752: 1481 / 1467; [2048 x 2048], f 5461:
    // 2929 / 2929; one of 19 sizes is slower, [2048 x 1024], f 2752, rank 64: 750 / 784, whose dU alone fills two whole rounds of
    // 64 x 64 tiles (rank 256: 924 / 913).
    const bool merge = c.bf16 ? bf16_plan_splits(both, bf.w.room, bf.w.parts_room) <
                                    0.95f * (bf16_plan_splits(alone, bf.w.room, bf.w.parts_room) +
                                             bf16_plan_splits(project, bf.w.room, 0))
                              : !f32_far(both);
    if (merge) {
      STAGE(MECEFO_STAGE_DGRAD_GATE_UP, s);
      both.clk = g_prof.cur_clk;
      if (!c.bf16 && kept) f32_plan_parts(both, bf.w.parts_room);
      return launch_store(c, bf, both, s, kept);
    }
  }
  TRY(dgrad(c, bf, Wg, Wu, dU, lddu, s, kept));
  if (q.n_lr == 0) return MECEFO_OK;
  STAGE(MECEFO_STAGE_PROJECT, s);
  project.clk = g_prof.cur_clk;
  if (c.bf16) bf16_plan_splits(project, bf.w.room, 0);
  return launch_store(c, bf, project, s);
}

// The weight gradients: exact ones, and Eq. (2) from the projections to the contraction over tokens.  Everything that
// reads dY and U is enqueued behind this.
mecefo_status_t wgrad_contract(const Ctx& c, const Bufs& bf, const LowRank& q, void* dW[3], int accumulate, hipStream_t s) {
  const int b = (int)c.b;
  if (q.n_ex > 0) {  // exact Wgrad: dW = Gy^T X, contraction over tokens
    STAGE(MECEFO_STAGE_WGRAD_EXACT, s);
    GemmLaunch g = new_launch(c, false, false, EPI_GRAD);
    g.nprob = q.n_ex;
    g.accumulate = accumulate;
    for (int j = 0; j < q.n_ex; ++j) {
      const int i = q.ex[j];
      g.p[j] = prob(q.Gy[i], nullptr, q.ldgy[i], q.X[i], nullptr, q.ldx[i], dW[i], nullptr, nullptr, q.lddw[i], q.m_out[i],
                    q.n_in[i], b, 1);
    }
    HIP_TRY(launch_gemm(g, s));
  }
  if (q.n_lr == 0) return MECEFO_OK;
  {  // contract over tokens: C = (Gy or X)^T T   [rows x r], K = b
    STAGE(MECEFO_STAGE_CONTRACT, s);
    GemmLaunch g = new_launch(c, false, false, EPI_STORE);
    g.nprob = q.n_lr;
    for (int j = 0; j < q.n_lr; ++j) {
      const int i = q.lr[j];
      g.p[j] = prob(q.in ? q.Gy[i] : q.X[i], nullptr, q.in ? q.ldgy[i] : q.ldx[i], q.T[i], nullptr, q.ldt[i], q.C[i],
                    nullptr, nullptr, q.ldt[i], q.in ? q.m_out[i] : q.n_in[i], q.P[i].r, b, 1);
    }
    // no more parts than the workspace holds
    if (b > 0) {
      if (c.bf16) bf16_plan_splits(g, bf.w.room, bf.w.parts_room);
      else f32_plan_splits(g, bf.w.splits);
    }
    TRY(launch_store(c, bf, g, s));
  }
  return MECEFO_OK;
}
// expand: dW = C P^T (SIDE_INPUT) or P C^T (SIDE_OUTPUT), K = r, into the gradient buffers, and a side job
mecefo_status_t wgrad_expand(const Ctx& c, const LowRank& q, void* dW[3], int accumulate, hipStream_t s,
                             const SideJob* side = nullptr) {
  GemmLaunch g = new_launch(c, true, true, EPI_GRAD);
  g.nprob = q.n_lr;
  g.accumulate = accumulate;
  for (int j = 0; j < q.n_lr; ++j) {
    const int i = q.lr[j];
    const mecefo_proj_t& P = q.P[i];
    g.p[j] = q.in ? prob(q.C[i], nullptr, q.ldt[i], P.P, nullptr, P.ld, dW[i], nullptr, nullptr, q.lddw[i], q.m_out[i],
                         q.n_in[i], P.r, 1)
                  : prob(P.P, nullptr, P.ld, q.C[i], nullptr, q.ldt[i], dW[i], nullptr, nullptr, q.lddw[i], q.m_out[i],
                         q.n_in[i], P.r, 1);
  }
  if (side) g.side = *side;
  if (q.n_lr > 0) {
    STAGE(MECEFO_STAGE_EXPAND, s);
    g.clk = g_prof.cur_clk;
    HIP_TRY(launch_gemm(g, s));
  }
  return dgamma_left(c, g, s);
}


// ---- standard-mode backward (Alg. 3, first branch) ----------------------------------------
struct FullWs {
  size_t dH, dQ, dK, dV, D, P, cs, sn, total;
  int64_t ldp;     // row stride of one [seq x seq] probability matrix
};

FullWs full_layout(const Ctx& c, const mecefo_attn_desc_t& a, size_t ffn_total) {
  FullWs w;
  size_t off = (size_t)up((int64_t)ffn_total, 256);
  auto take = [&](size_t bytes) { size_t o = off; off += (size_t)up((int64_t)bytes, 256); return o; };
  const size_t act_d = (size_t)c.b * c.dm * c.esz;
  w.ldp = up(a.seq, 8);
  w.dH = take(act_d);
  w.dQ = take(act_d);
  w.dK = take(act_d);
  w.dV = take(act_d);
  w.D = take((size_t)c.b * a.heads * 4);
  w.P = take((size_t)a.batch * a.heads * a.seq * w.ldp * c.esz);
  const int dh = c.dm / (a.heads > 0 ? a.heads : 1);
  w.cs = take((size_t)a.seq * (dh / 2) * 4);
  w.sn = take((size_t)a.seq * (dh / 2) * 4);
  w.total = off + 256;
  return w;
}

mecefo_status_t check_attn(const Ctx& c, const mecefo_attn_desc_t* a) {
  if (!a) return fail(MECEFO_ERR_INVALID_ARG, "attention descriptor is NULL");
  if (a->batch < 0 || a->seq < 0 || a->heads < 1) return fail(MECEFO_ERR_INVALID_ARG, "batch >= 0, seq >= 0, heads >= 1 required");
  if ((int64_t)a->batch * a->seq != c.b) return fail(MECEFO_ERR_INVALID_ARG, "batch * seq = %lld differs from tokens = %lld", (long long)a->batch * a->seq, (long long)c.b);
  if (c.dm % a->heads) return fail(MECEFO_ERR_INVALID_ARG, "d_model %d is not a multiple of heads %d", c.dm, a->heads);
  const int dh = c.dm / a->heads;
  if (dh % 2) return fail(MECEFO_ERR_INVALID_ARG, "head dimension %d must be even (rotary pairs)", dh);
  if (c.bf16 && dh % 8) return fail(MECEFO_ERR_UNSUPPORTED, "bf16 path needs a head dimension that is a multiple of 8 (got %d)", dh);
  if (c.dm > 16384) return fail(MECEFO_ERR_UNSUPPORTED, "d_model above 16384 is not built for the attention backward");
  if (a->ld_w_dd < c.dm) return fail(MECEFO_ERR_INVALID_ARG, "ld_w_dd is smaller than d_model");
  if (c.bf16 && a->ld_w_dd % 8) return fail(MECEFO_ERR_INVALID_ARG, "bf16 path needs ld_w_dd to be a multiple of 8");
  if (!(a->rope_theta > 0.f)) return fail(MECEFO_ERR_INVALID_ARG, "rope_theta must be positive");
  if ((int64_t)a->seq * up(a->seq, 8) * c.esz >= kMaxBytes || (int64_t)c.dm * a->ld_w_dd * 4 >= kMaxBytes)
    return fail(MECEFO_ERR_UNSUPPORTED, "a [seq x seq] score matrix or a [d x d] weight reaches 2 GiB");
  return MECEFO_OK;
}

// One batched attention product per (sequence, head): operands are token-major [b x d] tensors
// (head h at columns h*dh) or the [batch*heads][seq x ldp] probability buffer.
void per_head_tokens(const mecefo_attn_desc_t& a, int dh, int64_t ld, int64_t* bo, int64_t* bi) {
  *bo = (int64_t)a.seq * ld;
  *bi = dh;
}
void per_head_scores(const mecefo_attn_desc_t& a, int64_t ldp, int64_t* bo, int64_t* bi) {
  *bi = (int64_t)a.seq * ldp;
  *bo = *bi * a.heads;
}

// ---- block forward ------------------------------------------------------------------------
struct FwdWs {
  size_t Xn, rstd, Q, K, V, O, L, A, S32, P, cs, sn, total;
  int64_t ldp;
  int hc;        // heads per attention chunk
  bool fused;    // the attention kernel without scores; read from the switch once per public call
};

// The block forward takes the fused attention kernel (no score or probability buffer) whenever it is
// built for the shape; mecefo_set_option("attention", "gemm") keeps the materialised-score form for testing.  The
// workspace query and the call consult the same predicate.  The layout carries its answer: another host thread may
// change the switch during the call, and the regions behind the scores lie elsewhere in the other form.
bool fwd_attention_fused(const Ctx& c, const mecefo_attn_desc_t& a) {
  if (options().attn_gemm.load(std::memory_order_relaxed)) return false;
  // bf16 descriptors have row strides that are multiples of 8 (checked with the descriptor)
  return attn_fwd_fused_supported(c.bf16, c.dm / (a.heads > 0 ? a.heads : 1), a.seq > 0 ? a.seq : 1, 8);
}

FwdWs fwd_layout(const Ctx& c, const mecefo_attn_desc_t& a) {
  FwdWs w;
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off += (size_t)up((int64_t)bytes, 256); return o; };
  const size_t act_d = (size_t)c.b * c.dm * c.esz;
  const int dh = c.dm / (a.heads > 0 ? a.heads : 1);
  w.ldp = up(a.seq, 8);
  w.Xn = take(act_d);
  w.rstd = take((size_t)c.b * 4);
  w.Q = take(act_d); w.K = take(act_d); w.V = take(act_d); w.O = take(act_d);
  w.L = take((size_t)c.b * a.heads * 4);
  w.A = take((size_t)c.b * c.ldf * c.esz);
  // fp32 scores of one chunk of heads of one sequence: at most 256 MiB
  const int64_t per_head = (int64_t)a.seq * w.ldp * 4;
  int64_t hc = per_head > 0 ? ((int64_t)256 << 20) / per_head : a.heads;
  if (hc < 1) hc = 1;
  if (hc > a.heads) hc = a.heads;
  w.hc = (int)hc;
  w.fused = fwd_attention_fused(c, a);
  w.S32 = take(w.fused ? 0 : (size_t)hc * per_head);
  w.P = take(w.fused ? 0 : (size_t)hc * a.seq * w.ldp * c.esz);
  w.cs = take((size_t)a.seq * (dh / 2) * 4);
  w.sn = take((size_t)a.seq * (dh / 2) * 4);
  w.total = off + 256;
  return w;
}

// The block forward behind mecefo_block_fwd.  plan: the layout that every layer of one public call shares, NULL to
// make it here; tables_ready: the workspace holds the rotary tables of a previous layer of the same plan.
mecefo_status_t block_fwd(const mecefo_ffn_desc_t* desc, const mecefo_attn_desc_t* attn,
                          const mecefo_block_fwd_inputs_t* in, const mecefo_block_fwd_outputs_t* out,
                          const FwdWs* plan, void* ws, size_t ws_bytes, void* hip_stream, bool tables_ready);

mecefo_status_t check_lowrank_args(const Ctx& c, const mecefo_proj_t P[3], mecefo_side_t side, int exact_mask = 0) {
  if (side != MECEFO_SIDE_INPUT && side != MECEFO_SIDE_OUTPUT) return fail(MECEFO_ERR_INVALID_ARG, "side must be MECEFO_SIDE_INPUT or MECEFO_SIDE_OUTPUT");
  const bool in = side == MECEFO_SIDE_INPUT;
  if (!(exact_mask & 1)) TRY(check_proj(c, P[0], in ? c.dm : c.ff, "Pg"));
  if (!(exact_mask & 2)) TRY(check_proj(c, P[1], in ? c.dm : c.ff, "Pu"));
  if (!(exact_mask & 4)) TRY(check_proj(c, P[2], in ? c.ff : c.dm, "Pd"));
  return MECEFO_OK;
}

}  // namespace

// ---- scratch of the entry point that allocates nothing ------------------------------------
// Device memory that exists once per GPU from the moment the code object is loaded there.  In host code
// the name below stands for the symbol, not for an address: the address on the current device comes from
// hipGetSymbolAddress and is kept per device.
static __device__ __align__(256) unsigned char scratch[MECEFO_NOALLOC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::atomic<void*> g_scratch_ptr[kMaxDevices];

mecefo_status_t scratch_on_current_device(void** out) {
  int dev = 0;
  HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return fail(MECEFO_ERR_UNSUPPORTED, "device index %d is beyond the %d the scratch table holds", dev, kMaxDevices);
  void* p = g_scratch_ptr[dev].load(std::memory_order_acquire);
  if (!p) {   // several threads may resolve at once: every one of them gets the same address
    HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) return fail(MECEFO_ERR_LAUNCH, "hipGetSymbolAddress returned a NULL scratch address");
    g_scratch_ptr[dev].store(p, std::memory_order_release);
  }
  *out = p;
  return MECEFO_OK;
}
}  // namespace

extern "C" {

const char* mecefo_last_error(void) { return g_err; }
const char* mecefo_version(void) { return "mecefo-gfx950 0.2"; }

mecefo_status_t mecefo_init(void) {
  // bit i: prepared on device i (devices above 63 are prepared every time, kernel by kernel)
  static std::atomic<uint64_t> done{0};
  int dev = 0;
  HIP_TRY(hipGetDevice(&dev));
  const uint64_t bit = dev < 64 ? (uint64_t)1 << dev : 0;
  if (done.load(std::memory_order_acquire) & bit) return MECEFO_OK;
  HIP_TRY(prepare_gemm_bf16_nt());
  HIP_TRY(prepare_gemm_bf16_nn());
  HIP_TRY(prepare_gemm_bf16_tn());
  HIP_TRY(prepare_gemm_f32());
  HIP_TRY(prepare_attention_fwd());
  HIP_TRY(prepare_attention_bwd());
  void* p = nullptr;
  TRY(scratch_on_current_device(&p));
  done.fetch_or(bit, std::memory_order_release);
  return MECEFO_OK;
}

mecefo_status_t mecefo_set_option(const char* name, const char* value) {
  if (!name || !value) return fail(MECEFO_ERR_INVALID_ARG, "option name and value are required");
  if (!strcmp(name, "tile")) {
    for (int i = 0; i < kTileOptions; ++i)
      if (!strcmp(value, kTileOptionName[i])) { options().tile.store(i, std::memory_order_relaxed); return MECEFO_OK; }
    return fail(MECEFO_ERR_INVALID_ARG, "option tile: value must be auto, S, S4, T, T2, X, K, L4, L8R, L8 or LT (got %s)", value);
  }
  if (!strcmp(name, "attention")) {
    if (!strcmp(value, "auto")) { options().attn_gemm.store(0, std::memory_order_relaxed); return MECEFO_OK; }
    if (!strcmp(value, "gemm")) { options().attn_gemm.store(1, std::memory_order_relaxed); return MECEFO_OK; }
    return fail(MECEFO_ERR_INVALID_ARG, "option attention: value must be auto or gemm (got %s)", value);
  }
  return fail(MECEFO_ERR_INVALID_ARG, "unknown option %s", name);
}

mecefo_status_t mecefo_profile_enable(int max_launches) {
  if (max_launches < 1) return fail(MECEFO_ERR_INVALID_ARG, "max_launches must be >= 1");
  for (hipEvent_t e : g_prof.ev) (void)hipEventDestroy(e);
  g_prof.ev.assign((size_t)max_launches * 2, nullptr);
  g_prof.stage.assign((size_t)max_launches, 0);
  for (auto& e : g_prof.ev) HIP_TRY(hipEventCreate(&e));
  if (g_prof.clk) { (void)hipFree(g_prof.clk); g_prof.clk = nullptr; }
  const size_t clk_bytes = (size_t)max_launches * kClkPairs * 2 * sizeof(uint32_t);
  HIP_TRY(hipMalloc((void**)&g_prof.clk, clk_bytes));
  HIP_TRY(hipMemset(g_prof.clk, 0, clk_bytes));
  g_prof.used = 0;
  g_prof.on = true;
  return MECEFO_OK;
}

mecefo_status_t mecefo_profile_clock_mhz(double* mhz_by_stage) {
  if (!mhz_by_stage) return fail(MECEFO_ERR_INVALID_ARG, "output array is NULL");
  for (int i = 0; i < MECEFO_STAGE_COUNT; ++i) mhz_by_stage[i] = g_prof.mhz[i];
  return MECEFO_OK;
}

mecefo_status_t mecefo_profile_collect(double* ms_by_stage, int* launches_by_stage) {
  if (!ms_by_stage || !launches_by_stage) return fail(MECEFO_ERR_INVALID_ARG, "output arrays are NULL");
  for (int i = 0; i < MECEFO_STAGE_COUNT; ++i) { ms_by_stage[i] = 0.0; launches_by_stage[i] = 0; g_prof.mhz[i] = 0.0; }
  g_prof.on = false;
  g_prof.cur_clk = nullptr;
  for (size_t i = 0; i + 1 < g_prof.used; i += 2) {
    HIP_TRY(hipEventSynchronize(g_prof.ev[i + 1]));
    float ms = 0.f;
    HIP_TRY(hipEventElapsedTime(&ms, g_prof.ev[i], g_prof.ev[i + 1]));
    const int st = g_prof.stage[i / 2];
    ms_by_stage[st] += ms;
    launches_by_stage[st] += 1;
  }
  if (g_prof.clk && g_prof.used >= 2) {   // shader clock per stage: cycles / wall ticks (100 MHz) of the sampled workgroups
    const size_t launches = g_prof.used / 2;
    std::vector<uint32_t> h(launches * kClkPairs * 2);
    HIP_TRY(hipMemcpy(h.data(), g_prof.clk, h.size() * sizeof(uint32_t), hipMemcpyDeviceToHost));
    double cyc[MECEFO_STAGE_COUNT] = {}, ticks[MECEFO_STAGE_COUNT] = {};
    for (size_t l = 0; l < launches; ++l)
      for (int k = 0; k < kClkPairs; ++k) {
        const uint32_t c = h[(l * kClkPairs + k) * 2], w = h[(l * kClkPairs + k) * 2 + 1];
        if (c && w) { cyc[g_prof.stage[l]] += c; ticks[g_prof.stage[l]] += w; }
      }
    for (int i = 0; i < MECEFO_STAGE_COUNT; ++i) g_prof.mhz[i] = ticks[i] > 0 ? 100.0 * cyc[i] / ticks[i] : 0.0;
  }
  if (g_prof.clk) { (void)hipFree(g_prof.clk); g_prof.clk = nullptr; }
  for (hipEvent_t e : g_prof.ev) (void)hipEventDestroy(e);
  g_prof.ev.clear();
  g_prof.stage.clear();
  g_prof.used = 0;
  return MECEFO_OK;
}

mecefo_status_t mecefo_workspace_bytes(const mecefo_ffn_desc_t* desc, int r_gate, int r_up, int r_down,
                                       size_t* out_bytes) {
  Ctx c;
  TRY(check_desc(desc, &c));
  if (!out_bytes) return fail(MECEFO_ERR_INVALID_ARG, "out_bytes is NULL");
  if (r_gate < 0 || r_up < 0 || r_down < 0) return fail(MECEFO_ERR_INVALID_ARG, "ranks must be >= 0");
  const int r[3] = {r_gate, r_up, r_down};
  const size_t a = layout(c, r, MECEFO_SIDE_INPUT, 0, true).total;
  const size_t b2 = layout(c, r, MECEFO_SIDE_OUTPUT, 0, true).total;
  *out_bytes = a > b2 ? a : b2;
  return MECEFO_OK;
}

mecefo_status_t mecefo_ffn_fwd_recompute(const mecefo_ffn_desc_t* desc, const void* U, const void* Wg,
                                         const void* Wu, const void* Wd, void* G, void* Z, void* A, void* Y,
                                         void* ws, size_t ws_bytes, void* hip_stream) {
  (void)ws; (void)ws_bytes;
  Ctx c;
  TRY(check_desc(desc, &c));
  TRY(check_ptr(c, U, "U")); TRY(check_ptr(c, Wg, "Wg")); TRY(check_ptr(c, Wu, "Wu"));
  TRY(check_ptr(c, G, "G", false)); TRY(check_ptr(c, Z, "Z", false)); TRY(check_ptr(c, A, "A"));
  TRY(check_ptr(c, Y, "Y", false));
  if (Y) TRY(check_ptr(c, Wd, "Wd (needed for Y)"));
  hipStream_t s = (hipStream_t)hip_stream;
  const int b = (int)c.b;
  if (b == 0) return MECEFO_OK;
  const int pad = (int)(up(c.ff, 8) <= desc->ld_act_f ? up(c.ff, 8) : c.ff);
  {
    GemmLaunch g = new_launch(c, true, true, EPI_SWIGLU_FWD);
    g.nprob = 1;
    g.p[0] = prob(U, nullptr, desc->ld_act_d, Wg, Wu, desc->ld_w_fd, G, Z, A, desc->ld_act_f, b, c.ff, c.dm, 1, pad);
    HIP_TRY(launch_gemm(g, s));
  }
  if (Y) {  // Y = A Wd^T   [b x d], K = f
    GemmLaunch g = new_launch(c, true, true, EPI_STORE);
    g.nprob = 1;
    g.p[0] = prob(A, nullptr, desc->ld_act_f, Wd, nullptr, desc->ld_w_df, Y, nullptr, nullptr, desc->ld_act_d, b, c.dm, c.ff, 1);
    HIP_TRY(launch_gemm(g, s));
  }
  return MECEFO_OK;
}

mecefo_status_t mecefo_ffn_bwd_exact(const mecefo_ffn_desc_t* desc, const void* U, const void* dY,
                                     const void* Wg, const void* Wu, const void* Wd, const void* G,
                                     const void* Z, void* dU, void* dWg, void* dWu, void* dWd, int accumulate,
                                     void* ws, size_t ws_bytes, void* hip_stream) {
  Ctx c;
  TRY(check_desc(desc, &c));
  TRY(check_ptr(c, U, "U", c.b > 0)); TRY(check_ptr(c, dY, "dY", c.b > 0));
  TRY(check_ptr(c, Wg, "Wg")); TRY(check_ptr(c, Wu, "Wu")); TRY(check_ptr(c, Wd, "Wd"));
  if ((G == nullptr) != (Z == nullptr)) return fail(MECEFO_ERR_INVALID_ARG, "G and Z must both be given or both be NULL");
  TRY(check_ptr(c, G, "G", false)); TRY(check_ptr(c, Z, "Z", false)); TRY(check_ptr(c, dU, "dU", false));
  if (!dWg || !dWu || !dWd) return fail(MECEFO_ERR_INVALID_ARG, "dWg, dWu, dWd are required");
  if (c.bf16 && (((uintptr_t)dWg | (uintptr_t)dWu | (uintptr_t)dWd) % 16)) return fail(MECEFO_ERR_INVALID_ARG, "gradient buffers must be 16-byte aligned");
  const int r0[3] = {0, 0, 0};
  Bufs bf;
  TRY(carve(c, r0, MECEFO_SIDE_INPUT, ws, ws_bytes, &bf));
  hipStream_t s = (hipStream_t)hip_stream;
  TRY(recompute(c, bf, U, desc->ld_act_d, dY, desc->ld_act_d, Wg, Wu, Wd, G, Z, s));
  TRY(dgrad(c, bf, Wg, Wu, dU, desc->ld_act_d, s));
  // exact Wgrad: dWg = dG^T U, dWu = dZ^T U [f x d]; dWd = dY^T A [d x f]; contraction over tokens
  STAGE(MECEFO_STAGE_WGRAD_EXACT, s);
  GemmLaunch g = new_launch(c, false, false, EPI_GRAD);
  g.nprob = 3;
  g.accumulate = accumulate;
  const int b = (int)c.b;
  char* base = bf.base;
  g.p[0] = prob(base + bf.w.DG, nullptr, c.ldf, U, nullptr, desc->ld_act_d, dWg, nullptr, nullptr, desc->ld_w_fd, c.ff, c.dm, b, 1);
  g.p[1] = prob(base + bf.w.DZ, nullptr, c.ldf, U, nullptr, desc->ld_act_d, dWu, nullptr, nullptr, desc->ld_w_fd, c.ff, c.dm, b, 1);
  g.p[2] = prob(dY, nullptr, desc->ld_act_d, base + bf.w.AA, nullptr, c.ldf, dWd, nullptr, nullptr, desc->ld_w_df, c.dm, c.ff, b, 1);
  HIP_TRY(launch_gemm(g, s));
  return MECEFO_OK;
}

mecefo_status_t mecefo_ffn_bwd_lowrank(const mecefo_ffn_desc_t* desc, const void* U, const void* dY,
                                       const void* Wg, const void* Wu, const void* Wd, mecefo_proj_t Pg,
                                       mecefo_proj_t Pu, mecefo_proj_t Pd, mecefo_side_t side, void* dU,
                                       void* dWg, void* dWu, void* dWd, int accumulate, void* ws,
                                       size_t ws_bytes, void* hip_stream) {
  Ctx c;
  TRY(check_desc(desc, &c));
  TRY(check_ptr(c, U, "U", c.b > 0)); TRY(check_ptr(c, dY, "dY", c.b > 0));
  TRY(check_ptr(c, Wg, "Wg")); TRY(check_ptr(c, Wu, "Wu")); TRY(check_ptr(c, Wd, "Wd"));
  TRY(check_ptr(c, dU, "dU", false));
  if (!dWg || !dWu || !dWd) return fail(MECEFO_ERR_INVALID_ARG, "dWg, dWu, dWd are required");
  if (c.bf16 && (((uintptr_t)dWg | (uintptr_t)dWu | (uintptr_t)dWd) % 16)) return fail(MECEFO_ERR_INVALID_ARG, "gradient buffers must be 16-byte aligned");
  const mecefo_proj_t P[3] = {Pg, Pu, Pd};
  TRY(check_lowrank_args(c, P, side));
  const int r[3] = {Pg.r, Pu.r, Pd.r};
  Bufs bf;
  TRY(carve(c, r, side, ws, ws_bytes, &bf));
  hipStream_t s = (hipStream_t)hip_stream;
  const LowRank q = low_rank(c, bf, U, desc->ld_act_d, dY, desc->ld_act_d, P, side, 0);
  TRY(recompute(c, bf, U, desc->ld_act_d, dY, desc->ld_act_d, Wg, Wu, Wd, nullptr, nullptr, s));
  TRY(dgrad_and_project(c, bf, q, Wg, Wu, dU, desc->ld_act_d, s));
  void* dW[3] = {dWg, dWu, dWd};
  TRY(wgrad_contract(c, bf, q, dW, accumulate, s));
  return wgrad_expand(c, q, dW, accumulate, s);
}

mecefo_status_t mecefo_block_bwd_skip_ex(const mecefo_ffn_desc_t* desc, const void* H, const void* dOut,
                                         const void* gamma, const void* Wg, const void* Wu, const void* Wd,
                                         mecefo_proj_t Pg, mecefo_proj_t Pu, mecefo_proj_t Pd, mecefo_side_t side,
                                         const mecefo_skip_options_t* opt, void* dX, void* dgamma, void* dWg,
                                         void* dWu, void* dWd, int accumulate, void* ws, size_t ws_bytes,
                                         void* hip_stream) {
  Ctx c;
  TRY(check_desc(desc, &c));
  const void* Gs = opt ? opt->G : nullptr;
  const void* Zs = opt ? opt->Z : nullptr;
  const int exact_mask = opt ? opt->exact_wgrad_mask : 0;
  if (exact_mask & ~7) return fail(MECEFO_ERR_INVALID_ARG, "exact_wgrad_mask has bits beyond gate (1), up (2), down (4)");
  if ((Gs == nullptr) != (Zs == nullptr)) return fail(MECEFO_ERR_INVALID_ARG, "G and Z must both be given or both be NULL");
  TRY(check_ptr(c, Gs, "G", false)); TRY(check_ptr(c, Zs, "Z", false));
  TRY(check_ptr(c, H, "H", c.b > 0)); TRY(check_ptr(c, dOut, "dOut", c.b > 0)); TRY(check_ptr(c, gamma, "gamma", false));
  TRY(check_ptr(c, Wg, "Wg")); TRY(check_ptr(c, Wu, "Wu")); TRY(check_ptr(c, Wd, "Wd"));
  TRY(check_ptr(c, dX, "dX", c.b > 0));
  if (!dWg || !dWu || !dWd) return fail(MECEFO_ERR_INVALID_ARG, "dWg, dWu, dWd are required");
  if (c.bf16 && (((uintptr_t)dWg | (uintptr_t)dWu | (uintptr_t)dWd) % 16)) return fail(MECEFO_ERR_INVALID_ARG, "gradient buffers must be 16-byte aligned");
  if (dgamma && !gamma) return fail(MECEFO_ERR_INVALID_ARG, "dgamma requested but gamma is NULL");
  TRY(check_alias(dX, "dX", dOut, "dOut", act_span(c, desc->ld_act_d)));
  TRY(check_alias(dX, "dX", H, "H", act_span(c, desc->ld_act_d)));
  const mecefo_proj_t P[3] = {Pg, Pu, Pd};
  TRY(check_lowrank_args(c, P, side, exact_mask));
  const int r[3] = {(exact_mask & 1) ? 0 : Pg.r, (exact_mask & 2) ? 0 : Pu.r, (exact_mask & 4) ? 0 : Pd.r};
  Bufs bf;
  TRY(carve(c, r, side, ws, ws_bytes, &bf));
  hipStream_t s = (hipStream_t)hip_stream;
  char* base = bf.base;
  const void* U = H;
  int64_t ldu = desc->ld_act_d;
  const SideJob norm = norm_job(c, H, desc->ld_act_d, gamma, base + bf.w.U, (float*)(base + bf.w.rstd));
  const bool rides = gamma && c.b > 0 && norm_rides(c);
  if (gamma && c.b > 0) {  // recompute the norm output from the stored tensor
    if (!rides) TRY(norm_forward(c, norm, s));
    U = base + bf.w.U;
    ldu = c.dm;
  }
  void* dUb = base + bf.w.dU;
  const LowRank q = low_rank(c, bf, U, ldu, dOut, desc->ld_act_d, P, side, exact_mask);
  TRY(recompute(c, bf, U, ldu, dOut, desc->ld_act_d, Wg, Wu, Wd, Gs, Zs, s, rides ? &norm : nullptr));
  // Eq. (2) reads dOut (the down projection's output gradient) and, without a norm, H itself: when dX
  // is a buffer of its own the norm backward goes first, while dU is still in the caches; when dX overwrites dOut (or H)
  // it has to wait for the contraction, which needs the partial buffer.  The expand launch carries the sum of the gain
  // gradient.
  const bool dx_first = dX != dOut && dX != H;
  Parts parts;
  auto norm_args = [&]() {
    return norm_bwd_args(c, bf, bf.w, parts, H, desc->ld_act_d, gamma, dOut, desc->ld_act_d, dX, desc->ld_act_d, dgamma != nullptr);
  };
  const bool read_parts = gamma && c.b > 0 && norm_bwd_reads_parts(c, bf, norm_args());
  TRY(dgrad_and_project(c, bf, q, Wg, Wu, dUb, c.dm, s, read_parts ? &parts : nullptr));
  // Skip the MHA connection: the gradient handed to the previous layer is dH = dOut + normbwd(dU).
  SideJob later = {};
  auto norm_bwd = [&]() -> mecefo_status_t {
    if (gamma) return norm_backward(c, norm_args(), dgamma, accumulate, s, &later);
    STAGE(MECEFO_STAGE_NORM_BWD, s);
    if (c.b > 0) HIP_TRY(launch_add(c.bf16, dOut, desc->ld_act_d, dUb, c.dm, dX, desc->ld_act_d, c.b, c.dm, s));
    return MECEFO_OK;
  };
  if (dx_first) TRY(norm_bwd());
  void* dW[3] = {dWg, dWu, dWd};
  TRY(wgrad_contract(c, bf, q, dW, accumulate, s));
  if (!dx_first) TRY(norm_bwd());
  return wgrad_expand(c, q, dW, accumulate, s, &later);
}

mecefo_status_t mecefo_block_bwd_skip(const mecefo_ffn_desc_t* desc, const void* H, const void* dOut,
                                      const void* gamma, const void* Wg, const void* Wu, const void* Wd,
                                      mecefo_proj_t Pg, mecefo_proj_t Pu, mecefo_proj_t Pd, mecefo_side_t side,
                                      void* dX, void* dgamma, void* dWg, void* dWu, void* dWd, int accumulate,
                                      void* ws, size_t ws_bytes, void* hip_stream) {
  return mecefo_block_bwd_skip_ex(desc, H, dOut, gamma, Wg, Wu, Wd, Pg, Pu, Pd, side, nullptr, dX, dgamma, dWg, dWu,
                                  dWd, accumulate, ws, ws_bytes, hip_stream);
}

mecefo_status_t mecefo_block_full_workspace_bytes(const mecefo_ffn_desc_t* desc, const mecefo_attn_desc_t* attn,
                                                  size_t* out_bytes) {
  Ctx c;
  TRY(check_desc(desc, &c));
  TRY(check_attn(c, attn));
  if (!out_bytes) return fail(MECEFO_ERR_INVALID_ARG, "out_bytes is NULL");
  const int r0[3] = {0, 0, 0};
  *out_bytes = full_layout(c, *attn, layout(c, r0, MECEFO_SIDE_INPUT, 0, true).total).total;
  return MECEFO_OK;
}

mecefo_status_t mecefo_block_bwd_full(const mecefo_ffn_desc_t* desc, const mecefo_attn_desc_t* attn,
                                      const mecefo_block_inputs_t* in, const mecefo_block_grads_t* out,
                                      int accumulate, void* ws, size_t ws_bytes, void* hip_stream) {
  Ctx c;
  TRY(check_desc(desc, &c));
  TRY(check_attn(c, attn));
  if (!in || !out) return fail(MECEFO_ERR_INVALID_ARG, "input or output table is NULL");
  const bool any = c.b > 0;
  TRY(check_ptr(c, in->X, "X", any)); TRY(check_ptr(c, in->H, "H", any)); TRY(check_ptr(c, in->dOut, "dOut", any));
  TRY(check_ptr(c, in->g_attn, "g_attn")); TRY(check_ptr(c, in->g_ffn, "g_ffn"));
  TRY(check_ptr(c, in->Wq, "Wq")); TRY(check_ptr(c, in->Wk, "Wk")); TRY(check_ptr(c, in->Wv, "Wv")); TRY(check_ptr(c, in->Wo, "Wo"));
  TRY(check_ptr(c, in->Wg, "Wg")); TRY(check_ptr(c, in->Wu, "Wu")); TRY(check_ptr(c, in->Wd, "Wd"));
  TRY(check_ptr(c, in->Q, "Q", any)); TRY(check_ptr(c, in->K, "K", any)); TRY(check_ptr(c, in->V, "V", any)); TRY(check_ptr(c, in->O, "O", any));
  if (any && !in->L) return fail(MECEFO_ERR_INVALID_ARG, "L is NULL");
  TRY(check_ptr(c, out->dX, "dX", any));
  void* grads[9] = {out->dg_attn, out->dg_ffn, out->dWq, out->dWk, out->dWv, out->dWo, out->dWg, out->dWu, out->dWd};
  for (void* g : grads) {
    if (!g) return fail(MECEFO_ERR_INVALID_ARG, "every gradient buffer is required");
    if (c.bf16 && ((uintptr_t)g % 16)) return fail(MECEFO_ERR_INVALID_ARG, "gradient buffers must be 16-byte aligned");
  }
  const int r0[3] = {0, 0, 0};
  Workspace fw = layout(c, r0, MECEFO_SIDE_INPUT, 0, true);
  FullWs w = full_layout(c, *attn, fw.total);
  if (w.total > ws_bytes) {
    fw = layout(c, r0, MECEFO_SIDE_INPUT, 0, false);
    w = full_layout(c, *attn, fw.total);
  }
  if (w.total > ws_bytes) return fail(MECEFO_ERR_WORKSPACE_TOO_SMALL, "workspace has %zu bytes, %zu needed", ws_bytes, w.total);
  if (!ws) return fail(MECEFO_ERR_INVALID_ARG, "workspace is NULL");
  Bufs bf;
  bf.base = (char*)up((int64_t)(uintptr_t)ws, 256);
  bf.w = fw;
  char* base = bf.base;
  hipStream_t s = (hipStream_t)hip_stream;
  const mecefo_ffn_desc_t& d = *desc;
  const mecefo_attn_desc_t& a = *attn;
  const int b = (int)c.b, dm = c.dm, dh = dm / a.heads, S = a.seq;
  float* rstd = (float*)(base + fw.rstd);
  void* Ub = base + fw.U;       // norm(H), later norm(X)
  void* dUb = base + fw.dU;     // dU, later dO, later dXn
  void* dH = base + w.dH;
  void* dQ = base + w.dQ; void* dK = base + w.dK; void* dV = base + w.dV;
  float* D = (float*)(base + w.D);
  void* P = base + w.P;
  float* cs = (float*)(base + w.cs); float* sn = (float*)(base + w.sn);

  // ---- FFN module, exact: dH = dOut + normbwd(dU), dWg, dWu, dWd, dg_ffn
  const SideJob norm = norm_job(c, in->H, d.ld_act_d, in->g_ffn, Ub, rstd);
  const bool rides = any && norm_rides(c);
  if (any && !rides) TRY(norm_forward(c, norm, s));
  TRY(recompute(c, bf, Ub, dm, in->dOut, d.ld_act_d, in->Wg, in->Wu, in->Wd, nullptr, nullptr, s, rides ? &norm : nullptr));
  Parts parts;
  auto ffn_norm = [&]() {
    return norm_bwd_args(c, bf, fw, parts, in->H, d.ld_act_d, in->g_ffn, in->dOut, d.ld_act_d, dH, dm, true);
  };
  TRY(dgrad(c, bf, in->Wg, in->Wu, dUb, dm, s, any && norm_bwd_reads_parts(c, bf, ffn_norm()) ? &parts : nullptr));
  SideJob later = {};   // the sums of the gain gradients ride on the weight gradients' launches
  TRY(norm_backward(c, ffn_norm(), out->dg_ffn, accumulate, s, &later));
  GemmLaunch g = new_launch(c, false, false, EPI_GRAD);
  {
    STAGE(MECEFO_STAGE_WGRAD_EXACT, s);
    g.nprob = 3;
    g.accumulate = accumulate;
    g.side = later;
    g.clk = g_prof.cur_clk;
    g.p[0] = prob(base + fw.DG, nullptr, c.ldf, Ub, nullptr, dm, out->dWg, nullptr, nullptr, d.ld_w_fd, c.ff, dm, b, 1);
    g.p[1] = prob(base + fw.DZ, nullptr, c.ldf, Ub, nullptr, dm, out->dWu, nullptr, nullptr, d.ld_w_fd, c.ff, dm, b, 1);
    g.p[2] = prob(in->dOut, nullptr, d.ld_act_d, base + fw.AA, nullptr, c.ldf, out->dWd, nullptr, nullptr, d.ld_w_df, dm, c.ff, b, 1);
    HIP_TRY(launch_gemm(g, s));
  }
  TRY(dgamma_left(c, g, s));

  // ---- attention module
  if (any) {
    STAGE(MECEFO_STAGE_NORM_FWD, s);
    const RopeTables tables = {cs, sn, S, dh / 2, (double)a.rope_theta};
    HIP_TRY(launch_rmsnorm_fwd(c.bf16, in->X, d.ld_act_d, in->g_attn, d.rms_eps, Ub, dm, rstd, c.b, dm, s, &tables));
  }
  if (any) {  // dO = dH Wo  [b x d], K = d
    STAGE(MECEFO_STAGE_ATTN_OUT_BWD, s);
    GemmLaunch g = new_launch(c, true, false, EPI_STORE);
    g.nprob = 1;
    g.p[0] = prob(dH, nullptr, dm, in->Wo, nullptr, a.ld_w_dd, dUb, nullptr, nullptr, dm, b, dm, dm, 1);
    HIP_TRY(launch_gemm(g, s));
  }
  if (any) {
    const void* dO = dUb;
    const float scale = 1.0f / sqrtf((float)dh);
    int64_t tok_bo, tok_bi, ws_bo, ws_bi, sc_bo, sc_bi;
    per_head_tokens(a, dh, d.ld_act_d, &tok_bo, &tok_bi);   // caller tensors Q, K, V
    per_head_tokens(a, dh, dm, &ws_bo, &ws_bi);             // workspace tensors dO, dQ, dK, dV
    per_head_scores(a, w.ldp, &sc_bo, &sc_bi);
    auto batched = [&](GemmProblem& p, int64_t abo, int64_t abi, int64_t bbo, int64_t bbi, int64_t cbo, int64_t cbi) {
      p.batch = a.batch * a.heads;
      p.batch_inner = a.heads;
      p.a_bo = abo; p.a_bi = abi; p.b_bo = bbo; p.b_bi = bbi; p.c_bo = cbo; p.c_bi = cbi;
    };
    {
      STAGE(MECEFO_STAGE_ATTN_ROWDOT, s);
      HIP_TRY(launch_attn_rowdot(c.bf16, dO, dm, in->O, d.ld_act_d, D, c.b, S, a.heads, dh, s));
    }
    // mecefo_set_option("attention", "gemm") forces the five-product form
    const bool fused = attn_bwd_fused_supported(c.bf16, dh, S, w.ldp) && !options().attn_gemm.load(std::memory_order_relaxed);
    if (fused) {  // dK, dV and dS in one kernel; P stays in registers
      STAGE(MECEFO_STAGE_ATTN_FUSED_KV, s);
      HIP_TRY(launch_attn_bwd_kv(in->Q, in->K, in->V, d.ld_act_d, dO, dK, dV, dm, in->L, D, P, w.ldp, a.batch, S,
                                 a.heads, dh, scale, s));
    }
    if (!fused) {
      {  // P = exp(scale Q K^T - L) below the diagonal, 0 above
        STAGE(MECEFO_STAGE_ATTN_PROBS, s);
        GemmLaunch g = new_launch(c, true, true, EPI_ATTN_P);
        g.nprob = 1;
        g.p[0] = prob(in->Q, nullptr, d.ld_act_d, in->K, nullptr, d.ld_act_d, P, nullptr, nullptr, w.ldp, S, S, dh, 1);
        batched(g.p[0], tok_bo, tok_bi, tok_bo, tok_bi, sc_bo, sc_bi);
        g.p[0].rowvec = in->L; g.p[0].scale = scale; g.p[0].causal = CAUSAL_TILE;
        HIP_TRY(launch_gemm(g, s));
      }
      {  // dV = P^T dO   [seq x dh], contraction over the query index
        STAGE(MECEFO_STAGE_ATTN_DV, s);
        GemmLaunch g = new_launch(c, false, false, EPI_STORE);
        g.nprob = 1;
        g.p[0] = prob(P, nullptr, w.ldp, dO, nullptr, dm, dV, nullptr, nullptr, dm, S, dh, S, 1);
        batched(g.p[0], sc_bo, sc_bi, ws_bo, ws_bi, ws_bo, ws_bi);
        g.p[0].causal = CAUSAL_K_FROM_M;
        HIP_TRY(launch_gemm(g, s));
      }
      {  // dS = P * (dO V^T - D) * scale, in place on P
        STAGE(MECEFO_STAGE_ATTN_DS, s);
        GemmLaunch g = new_launch(c, true, true, EPI_ATTN_DS);
        g.nprob = 1;
        g.p[0] = prob(dO, nullptr, dm, in->V, nullptr, d.ld_act_d, P, nullptr, nullptr, w.ldp, S, S, dh, 1);
        batched(g.p[0], ws_bo, ws_bi, tok_bo, tok_bi, sc_bo, sc_bi);
        g.p[0].rowvec = D; g.p[0].scale = scale; g.p[0].causal = CAUSAL_TILE;
        HIP_TRY(launch_gemm(g, s));
      }
    }
    {  // dQ = dS K   [seq x dh], contraction over the key index
      STAGE(MECEFO_STAGE_ATTN_DQ, s);
      GemmLaunch g = new_launch(c, true, false, EPI_STORE);
      g.nprob = 1;
      g.p[0] = prob(P, nullptr, w.ldp, in->K, nullptr, d.ld_act_d, dQ, nullptr, nullptr, dm, S, dh, S, 1);
      batched(g.p[0], sc_bo, sc_bi, tok_bo, tok_bi, ws_bo, ws_bi);
      g.p[0].causal = CAUSAL_K_UPTO_M;
      HIP_TRY(launch_gemm(g, s));
    }
    if (!fused) {  // dK = dS^T Q   [seq x dh], contraction over the query index
      STAGE(MECEFO_STAGE_ATTN_DK, s);
      GemmLaunch g = new_launch(c, false, false, EPI_STORE);
      g.nprob = 1;
      g.p[0] = prob(P, nullptr, w.ldp, in->Q, nullptr, d.ld_act_d, dK, nullptr, nullptr, dm, S, dh, S, 1);
      batched(g.p[0], sc_bo, sc_bi, tok_bo, tok_bi, ws_bo, ws_bi);
      g.p[0].causal = CAUSAL_K_FROM_M;
      HIP_TRY(launch_gemm(g, s));
    }
    {
      STAGE(MECEFO_STAGE_ROPE_BWD, s);
      HIP_TRY(launch_rope(c.bf16, dQ, dK, dm, cs, sn, c.b, S, a.heads, dh, true, s));
    }
  }
  // dWq, dWk, dWv = (dQ, dK, dV)^T Xn and dWo = dH^T O, all [d x d], K = tokens: one launch fills the chip where three and
  // one leave parts of it idle (2048 tokens, d 2048: 256 tiles of 256 x 256, 82 us instead of 71 and 34).
  auto wgrads = [&](const SideJob& side) -> mecefo_status_t {
    GemmLaunch g = new_launch(c, false, false, EPI_GRAD);
    g.nprob = 4;
    g.accumulate = accumulate;
    g.side = side;
    void* dst[3] = {out->dWq, out->dWk, out->dWv};
    const void* src[3] = {dQ, dK, dV};
    for (int i = 0; i < 3; ++i)
      g.p[i] = prob(src[i], nullptr, dm, Ub, nullptr, dm, dst[i], nullptr, nullptr, a.ld_w_dd, dm, dm, b, 1);
    g.p[3] = prob(dH, nullptr, dm, in->O, nullptr, d.ld_act_d, out->dWo, nullptr, nullptr, a.ld_w_dd, dm, dm, b, 1);
    {
      STAGE(MECEFO_STAGE_QKV_WGRAD, s);
      g.clk = g_prof.cur_clk;
      HIP_TRY(launch_gemm(g, s));
    }
    return dgamma_left(c, g, s);
  };
  // The sum of the gain gradient rides on them, behind the norm backward; a dX that lies over O is written when O was read.
  const uintptr_t x0 = (uintptr_t)out->dX, o0 = (uintptr_t)in->O, span = (uintptr_t)(c.b * d.ld_act_d * c.esz);
  const bool dx_last = x0 < o0 + span && o0 < x0 + span;
  if (dx_last) TRY(wgrads(SideJob{}));
  parts = Parts();
  auto attn_norm = [&]() {
    return norm_bwd_args(c, bf, fw, parts, in->X, d.ld_act_d, in->g_attn, dH, dm, out->dX, d.ld_act_d, true);
  };
  if (any) {  // dXn = dQ Wq + dK Wk + dV Wv   [b x d], three K segments of length d
    STAGE(MECEFO_STAGE_QKV_DGRAD, s);
    GemmLaunch g = new_launch(c, true, false, EPI_STORE);
    g.nprob = 1;
    g.p[0] = prob(dQ, dK, dm, in->Wq, in->Wk, a.ld_w_dd, dUb, nullptr, nullptr, dm, b, dm, dm, 3);
    g.p[0].A[2] = dV; g.p[0].B[2] = in->Wv;
    if (norm_bwd_reads_parts(c, bf, attn_norm())) {
      g.p[0].read_parts = true;
      if (c.bf16) bf16_plan_splits(g, fw.room, fw.parts_room);
      else f32_plan_parts(g, fw.parts_room);
    }
    TRY(launch_store(c, bf, g, s, &parts));
  }
  // dX = dH + normbwd(dXn), dg_attn
  later = SideJob{};
  TRY(norm_backward(c, attn_norm(), out->dg_attn, accumulate, s, dx_last ? nullptr : &later));
  return dx_last ? MECEFO_OK : wgrads(later);
}

mecefo_status_t mecefo_block_fwd_workspace_bytes(const mecefo_ffn_desc_t* desc, const mecefo_attn_desc_t* attn,
                                                 size_t* out_bytes) {
  Ctx c;
  TRY(check_desc(desc, &c));
  TRY(check_attn(c, attn));
  if (!out_bytes) return fail(MECEFO_ERR_INVALID_ARG, "out_bytes is NULL");
  *out_bytes = fwd_layout(c, *attn).total;
  return MECEFO_OK;
}

mecefo_status_t mecefo_block_fwd(const mecefo_ffn_desc_t* desc, const mecefo_attn_desc_t* attn,
                                 const mecefo_block_fwd_inputs_t* in, const mecefo_block_fwd_outputs_t* out,
                                 void* ws, size_t ws_bytes, void* hip_stream) {
  return block_fwd(desc, attn, in, out, nullptr, ws, ws_bytes, hip_stream, false);
}

}  // extern "C"

namespace {
mecefo_status_t block_fwd(const mecefo_ffn_desc_t* desc, const mecefo_attn_desc_t* attn,
                          const mecefo_block_fwd_inputs_t* in, const mecefo_block_fwd_outputs_t* out,
                          const FwdWs* plan, void* ws, size_t ws_bytes, void* hip_stream, bool tables_ready) {
  Ctx c;
  TRY(check_desc(desc, &c));
  TRY(check_attn(c, attn));
  if (!in || !out) return fail(MECEFO_ERR_INVALID_ARG, "input or output table is NULL");
  const bool any = c.b > 0;
  TRY(check_ptr(c, in->X, "X", any));
  TRY(check_ptr(c, in->g_attn, "g_attn")); TRY(check_ptr(c, in->g_ffn, "g_ffn"));
  TRY(check_ptr(c, in->Wq, "Wq")); TRY(check_ptr(c, in->Wk, "Wk")); TRY(check_ptr(c, in->Wv, "Wv")); TRY(check_ptr(c, in->Wo, "Wo"));
  TRY(check_ptr(c, in->Wg, "Wg")); TRY(check_ptr(c, in->Wu, "Wu")); TRY(check_ptr(c, in->Wd, "Wd"));
  TRY(check_ptr(c, out->Out, "Out", any)); TRY(check_ptr(c, out->H, "H", any));
  const int given = (out->Q != nullptr) + (out->K != nullptr) + (out->V != nullptr) + (out->O != nullptr) + (out->L != nullptr);
  if (given != 0 && given != 5) return fail(MECEFO_ERR_INVALID_ARG, "Q, K, V, O, L must all be given (standard mode) or all be NULL (neighbor mode)");
  TRY(check_ptr(c, out->Q, "Q", false)); TRY(check_ptr(c, out->K, "K", false)); TRY(check_ptr(c, out->V, "V", false)); TRY(check_ptr(c, out->O, "O", false));
  if (any && out->Out == in->X) return fail(MECEFO_ERR_INVALID_ARG, "Out must not alias X");
  const FwdWs w = plan ? *plan : fwd_layout(c, *attn);
  if (w.total > ws_bytes) return fail(MECEFO_ERR_WORKSPACE_TOO_SMALL, "workspace has %zu bytes, %zu needed", ws_bytes, w.total);
  if (!ws) return fail(MECEFO_ERR_INVALID_ARG, "workspace is NULL");
  if (!any) return MECEFO_OK;
  char* base = (char*)up((int64_t)(uintptr_t)ws, 256);
  hipStream_t s = (hipStream_t)hip_stream;
  const mecefo_ffn_desc_t& d = *desc;
  const mecefo_attn_desc_t& a = *attn;
  const int b = (int)c.b, dm = c.dm, dh = dm / a.heads, S = a.seq;
  const bool keep = given == 5;
  void* Xn = base + w.Xn;
  float* rstd = (float*)(base + w.rstd);
  void* Q = keep ? out->Q : base + w.Q; void* K = keep ? out->K : base + w.K;
  void* V = keep ? out->V : base + w.V; void* O = keep ? out->O : base + w.O;
  float* L = keep ? out->L : (float*)(base + w.L);
  const int64_t ldq = keep ? d.ld_act_d : dm;   // row stride of Q, K, V, O
  float* cs = (float*)(base + w.cs); float* sn = (float*)(base + w.sn);
  float* S32 = (float*)(base + w.S32);
  void* P = base + w.P;

  const RopeTables tables = {cs, sn, S, dh / 2, (double)a.rope_theta};
  HIP_TRY(launch_rmsnorm_fwd(c.bf16, in->X, d.ld_act_d, in->g_attn, d.rms_eps, Xn, dm, rstd, c.b, dm, s, tables_ready ? nullptr : &tables));
  {  // Q, K, V = Xn Wq^T, Xn Wk^T, Xn Wv^T  [b x d], K = d; Q and K rotated in the epilogue where its waves hold whole heads
    GemmLaunch g = new_launch(c, true, true, EPI_STORE);
    g.nprob = 3;
    void* dst[3] = {Q, K, V};
    const void* wt[3] = {in->Wq, in->Wk, in->Wv};
    for (int i = 0; i < 3; ++i) g.p[i] = prob(Xn, nullptr, dm, wt[i], nullptr, a.ld_w_dd, dst[i], nullptr, nullptr, ldq, b, dm, dm, 1);
    g.tile = c.bf16 ? gemm_bf16_rope_tile(g, dh) : -1;
    const bool rotate = g.tile >= 0;
    if (rotate) {
      g.epi = EPI_ROPE;
      for (int i = 0; i < 2; ++i) { g.p[i].rope_half = dh / 2; g.p[i].rope_seq = S; g.p[i].rowvec = cs; g.p[i].addend = sn; }
    }
    HIP_TRY(launch_gemm(g, s));
    if (!rotate) {
      HIP_TRY(launch_rope(c.bf16, Q, K, ldq, cs, sn, c.b, S, a.heads, dh, false, s));
    }
  }
  const float scale = 1.0f / sqrtf((float)dh);
  if (w.fused) HIP_TRY(launch_attn_fwd(Q, K, V, O, ldq, L, a.batch, S, a.heads, dh, scale, s));
  for (int bi = 0; bi < (w.fused ? 0 : a.batch); ++bi)
    for (int h0 = 0; h0 < a.heads; h0 += w.hc) {
      const int hc = a.heads - h0 < w.hc ? a.heads - h0 : w.hc;
      const int64_t tok = ((int64_t)bi * S * ldq + (int64_t)h0 * dh) * c.esz;
      const char* Qc = (const char*)Q + tok; const char* Kc = (const char*)K + tok; const char* Vc = (const char*)V + tok;
      char* Oc = (char*)O + tok;
      auto batched = [&](GemmProblem& p, int64_t abi, int64_t bbi, int64_t cbi) {
        p.batch = hc; p.batch_inner = hc;
        p.a_bo = 0; p.b_bo = 0; p.c_bo = 0; p.a_bi = abi; p.b_bi = bbi; p.c_bi = cbi;
      };
      {  // raw scores q.k in fp32, blocks above the diagonal skipped
        GemmLaunch g = new_launch(c, true, true, EPI_GRAD);
        g.out_f32 = true;
        g.nprob = 1;
        g.p[0] = prob(Qc, nullptr, ldq, Kc, nullptr, ldq, S32, nullptr, nullptr, w.ldp, S, S, dh, 1);
        // output offsets are counted in operand elements: fp32 scores behind bf16 operands take two each
        batched(g.p[0], dh, dh, (int64_t)S * w.ldp * (c.bf16 ? 2 : 1));
        g.p[0].causal = CAUSAL_TILE;
        HIP_TRY(launch_gemm(g, s));
      }
      HIP_TRY(launch_softmax_rows(c.bf16, S32, w.ldp, P, w.ldp, L + ((int64_t)bi * a.heads + h0) * S, hc, S, scale, s));
      {  // O = P V  [seq x dh], contraction over the keys up to the diagonal block
        GemmLaunch g = new_launch(c, true, false, EPI_STORE);
        g.nprob = 1;
        g.p[0] = prob(P, nullptr, w.ldp, Vc, nullptr, ldq, Oc, nullptr, nullptr, ldq, S, dh, S, 1);
        batched(g.p[0], (int64_t)S * w.ldp, dh, dh);
        g.p[0].causal = CAUSAL_K_UPTO_M;
        HIP_TRY(launch_gemm(g, s));
      }
    }
  {  // H = X + O Wo^T
    GemmLaunch g = new_launch(c, true, true, EPI_RESID);
    g.nprob = 1;
    g.p[0] = prob(O, nullptr, ldq, in->Wo, nullptr, a.ld_w_dd, out->H, const_cast<void*>(in->X), nullptr, d.ld_act_d, b, dm, dm, 1);
    HIP_TRY(launch_gemm(g, s));
  }
  // FFN: U = norm(H), A = silu(U Wg^T) * (U Wu^T), Out = H + A Wd^T
  HIP_TRY(launch_rmsnorm_fwd(c.bf16, out->H, d.ld_act_d, in->g_ffn, d.rms_eps, Xn, dm, rstd, c.b, dm, s));
  void* AA = base + w.A;
  {
    GemmLaunch g = new_launch(c, true, true, EPI_SWIGLU_FWD);
    g.nprob = 1;
    g.p[0] = prob(Xn, nullptr, dm, in->Wg, in->Wu, d.ld_w_fd, nullptr, nullptr, AA, c.ldf, b, c.ff, dm, 1, (int)c.ldf);
    HIP_TRY(launch_gemm(g, s));
  }
  {
    GemmLaunch g = new_launch(c, true, true, EPI_RESID);
    g.nprob = 1;
    g.p[0] = prob(AA, nullptr, c.ldf, in->Wd, nullptr, d.ld_w_df, out->Out, out->H, nullptr, d.ld_act_d, b, dm, c.ff, 1);
    HIP_TRY(launch_gemm(g, s));
  }
  return MECEFO_OK;
}
}  // namespace

extern "C" {

mecefo_status_t mecefo_stack_workspace_bytes(const mecefo_ffn_desc_t* desc, const mecefo_attn_desc_t* attn,
                                             int r_gate, int r_up, int r_down, size_t* out_bytes) {
  size_t fwd = 0, bwd = 0;
  TRY(mecefo_block_fwd_workspace_bytes(desc, attn, &fwd));
  TRY(mecefo_workspace_bytes(desc, r_gate, r_up, r_down, &bwd));
  if (!out_bytes) return fail(MECEFO_ERR_INVALID_ARG, "out_bytes is NULL");
  // two [b x ld] activation buffers for the forward ping-pong behind the larger of the two workspaces
  const size_t act = (size_t)up((int64_t)desc->tokens * desc->ld_act_d * (desc->dtype == MECEFO_BF16 ? 2 : 4), 256);
  *out_bytes = (fwd > bwd ? fwd : bwd) + 2 * act + 512;
  return MECEFO_OK;
}

mecefo_status_t mecefo_stack_fwd_neighbor(const mecefo_ffn_desc_t* desc, const mecefo_attn_desc_t* attn,
                                          int n_layers, const mecefo_layer_weights_t* layers, const void* X0,
                                          void* const* H, void* X_out, void* ws, size_t ws_bytes,
                                          void* hip_stream) {
  Ctx c;
  TRY(check_desc(desc, &c));
  TRY(check_attn(c, attn));
  if (n_layers < 1) return fail(MECEFO_ERR_INVALID_ARG, "n_layers must be >= 1");
  if (!layers || !H) return fail(MECEFO_ERR_INVALID_ARG, "layers and H are required");
  if (c.b > 0 && X_out == X0) return fail(MECEFO_ERR_INVALID_ARG, "X_out must not alias X0");
  const FwdWs plan = fwd_layout(c, *attn);
  const size_t inner = plan.total;
  const size_t act = (size_t)up(c.b * desc->ld_act_d * c.esz, 256);
  if (!ws) return fail(MECEFO_ERR_INVALID_ARG, "workspace is NULL");
  char* base = (char*)up((int64_t)(uintptr_t)ws, 256);
  const size_t lead = (size_t)(base - (char*)ws);
  if (lead + 2 * act + inner > ws_bytes) return fail(MECEFO_ERR_WORKSPACE_TOO_SMALL, "workspace has %zu bytes, %zu needed", ws_bytes, lead + 2 * act + inner);
  void* pp[2] = {base, base + act};
  void* inner_ws = base + 2 * act;
  const void* x = X0;
  for (int l = 0; l < n_layers; ++l) {
    const mecefo_layer_weights_t& w = layers[l];
    mecefo_block_fwd_inputs_t in = {x, w.g_attn, w.g_ffn, w.Wq, w.Wk, w.Wv, w.Wo, w.Wg, w.Wu, w.Wd};
    void* y = l == n_layers - 1 ? X_out : pp[l & 1];
    mecefo_block_fwd_outputs_t out = {y, H[l], nullptr, nullptr, nullptr, nullptr, nullptr};
    // every layer of the call uses the same workspace and layout: the angle tables of the first one serve them all
    mecefo_status_t st = block_fwd(desc, attn, &in, &out, &plan, inner_ws, ws_bytes - lead - 2 * act, hip_stream, l > 0);
    if (st != MECEFO_OK) return st;
    x = y;
  }
  return MECEFO_OK;
}

mecefo_status_t mecefo_stack_bwd_skip(const mecefo_ffn_desc_t* desc, int n_layers, const mecefo_layer_weights_t* layers,
                                      const void* const* H, const mecefo_layer_lowrank_t* lowrank, mecefo_side_t side,
                                      const void* dOut_top, void* dX_bottom, int accumulate, void* ws,
                                      size_t ws_bytes, void* hip_stream) {
  if (n_layers < 1) return fail(MECEFO_ERR_INVALID_ARG, "n_layers must be >= 1");
  if (!layers || !H || !lowrank) return fail(MECEFO_ERR_INVALID_ARG, "layers, H and lowrank are required");
  // the gradient travels down in dX_bottom's buffer: every layer overwrites its dOut with its dX
  const void* g = dOut_top;
  for (int l = n_layers - 1; l >= 0; --l) {
    const mecefo_layer_weights_t& w = layers[l];
    const mecefo_layer_lowrank_t& q = lowrank[l];
    mecefo_status_t st = mecefo_block_bwd_skip(desc, H[l], g, w.g_ffn, w.Wg, w.Wu, w.Wd, q.Pg, q.Pu, q.Pd, side,
                                               dX_bottom, q.dg_ffn, q.dWg, q.dWu, q.dWd, accumulate, ws, ws_bytes,
                                               hip_stream);
    if (st != MECEFO_OK) return st;
    g = dX_bottom;
  }
  return MECEFO_OK;
}


mecefo_status_t mecefo_block_bwd_skip_noalloc(const mecefo_ffn_desc_t* desc, const void* H, const void* dOut,
                                              const void* gamma, const void* Wg, const void* Wu, const void* Wd,
                                              mecefo_proj_t Pg, mecefo_proj_t Pu, mecefo_proj_t Pd, mecefo_side_t side,
                                              void* dX, void* dgamma, void* dWg, void* dWu, void* dWd, int accumulate,
                                              void* hip_stream) {
  Ctx c;
  TRY(check_desc(desc, &c));
  const int r[3] = {Pg.r > 0 ? Pg.r : 0, Pu.r > 0 ? Pu.r : 0, Pd.r > 0 ? Pd.r : 0};
  const size_t in = layout(c, r, MECEFO_SIDE_INPUT, 0, false).total, other = layout(c, r, MECEFO_SIDE_OUTPUT, 0, false).total;
  const size_t need = in > other ? in : other;
  if (need > (size_t)MECEFO_NOALLOC_SCRATCH_BYTES)
    return fail(MECEFO_ERR_WORKSPACE_TOO_SMALL,
                "this shape needs %zu bytes of scratch; the static buffer of mecefo_block_bwd_skip_noalloc holds %zu "
                "(use mecefo_block_bwd_skip with a workspace of the caller's)", need, (size_t)MECEFO_NOALLOC_SCRATCH_BYTES);
  void* ws = nullptr;
  TRY(scratch_on_current_device(&ws));
  // Nothing in the scratch has to start at zero: every region of the workspace layout is written by a
  // kernel of this call before a later kernel of the same call reads it.
  return mecefo_block_bwd_skip(desc, H, dOut, gamma, Wg, Wu, Wd, Pg, Pu, Pd, side, dX, dgamma, dWg, dWu, dWd, accumulate,
                               ws, (size_t)MECEFO_NOALLOC_SCRATCH_BYTES, hip_stream);
}

// ---- Alg. 1 / Alg. 3 bookkeeping and the stack backward with a mode per layer ----------------
int mecefo_refresh_due(int64_t t, int64_t tau) { return tau >= 1 && t >= 0 && t % tau == 0; }

void mecefo_counters_reset(int64_t* t, int n_layers) {
  if (!t) return;
  for (int l = 0; l < n_layers; ++l) t[l] = 0;
}

mecefo_status_t mecefo_stack_mixed_workspace_bytes(const mecefo_ffn_desc_t* desc, const mecefo_attn_desc_t* attn,
                                                   int r_gate, int r_up, int r_down, size_t* out_bytes) {
  size_t full = 0, skip = 0;
  TRY(mecefo_block_full_workspace_bytes(desc, attn, &full));
  TRY(mecefo_workspace_bytes(desc, r_gate, r_up, r_down, &skip));
  if (!out_bytes) return fail(MECEFO_ERR_INVALID_ARG, "out_bytes is NULL");
  size_t best = full > skip ? full : skip;
  // projection refresh of the three FFN matrices, one after the other in the same workspace (either side)
  const int rr[3] = {r_gate, r_up, r_down};
  for (int i = 0; i < 3; ++i) {
    if (rr[i] <= 0) continue;
    const int m = i < 2 ? desc->d_ff : desc->d_model, n = i < 2 ? desc->d_model : desc->d_ff;
    for (int left = 0; left < 2; ++left) {
      size_t pw = 0;
      TRY(mecefo_projection_workspace_bytes(desc->dtype, m, n, rr[i], left, &pw));
      if (pw > best) best = pw;
    }
  }
  *out_bytes = best;
  return MECEFO_OK;
}

mecefo_status_t mecefo_stack_bwd_mixed(const mecefo_ffn_desc_t* desc, const mecefo_attn_desc_t* attn, int n_layers,
                                       const mecefo_mode_t* modes, const mecefo_block_inputs_t* in,
                                       const mecefo_block_grads_t* grads, const mecefo_layer_lowrank_t* lowrank,
                                       mecefo_side_t side, const mecefo_refresh_policy_t* policy, int64_t* t,
                                       const void* dOut_top, void* dX_bottom, int accumulate, void* ws,
                                       size_t ws_bytes, void* hip_stream) {
  if (n_layers < 1) return fail(MECEFO_ERR_INVALID_ARG, "n_layers must be >= 1");
  if (!modes || !in || !grads) return fail(MECEFO_ERR_INVALID_ARG, "modes, in and grads are required");
  if (!desc) return fail(MECEFO_ERR_INVALID_ARG, "descriptor is NULL");
  bool any_neighbor = false;
  for (int l = 0; l < n_layers; ++l) {
    if (modes[l] != MECEFO_MODE_STANDARD && modes[l] != MECEFO_MODE_NEIGHBOR)
      return fail(MECEFO_ERR_INVALID_ARG, "layer %d: mode must be MECEFO_MODE_STANDARD or MECEFO_MODE_NEIGHBOR", l);
    any_neighbor |= modes[l] == MECEFO_MODE_NEIGHBOR;
  }
  if (any_neighbor && !lowrank) return fail(MECEFO_ERR_INVALID_ARG, "lowrank is required when a layer runs in neighbor mode");
  if ((policy == nullptr) != (t == nullptr)) return fail(MECEFO_ERR_INVALID_ARG, "policy and t must both be given or both be NULL");
  if (policy && (policy->tau < 1 || policy->power_iters < 1 || policy->cond_steps < 0 || policy->polish_steps < 0))
    return fail(MECEFO_ERR_INVALID_ARG, "refresh policy: tau >= 1, power_iters >= 1, cond_steps >= 0, polish_steps >= 0 required");
  const bool left = side == MECEFO_SIDE_OUTPUT;
  // the gradient travels down in dX_bottom's buffer: every layer overwrites its dOut with its dX
  const void* g = dOut_top;
  for (int l = n_layers - 1; l >= 0; --l) {
    const mecefo_block_inputs_t& x = in[l];
    const mecefo_block_grads_t& o = grads[l];
    mecefo_status_t st;
    if (modes[l] == MECEFO_MODE_STANDARD) {           // Alg. 3, first branch: exact gradients, MHA included
      mecefo_block_inputs_t xi = x;
      xi.dOut = g;
      mecefo_block_grads_t oi = o;
      oi.dX = dX_bottom;
      st = mecefo_block_bwd_full(desc, attn, &xi, &oi, accumulate, ws, ws_bytes, hip_stream);
    } else {                                          // neighbor branch
      const mecefo_layer_lowrank_t& q = lowrank[l];
      if (policy && mecefo_refresh_due(t[l], policy->tau)) {
        // V1 of the current weights (Alg. 3: every tau neighbor steps of this layer), warm-started from and
        // written over the layer's present projection
        const void* W[3] = {x.Wg, x.Wu, x.Wd};
        const mecefo_proj_t P[3] = {q.Pg, q.Pu, q.Pd};
        for (int i = 0; i < 3; ++i) {
          const int m = i < 2 ? desc->d_ff : desc->d_model, n = i < 2 ? desc->d_model : desc->d_ff;
          const int64_t ldw = i < 2 ? desc->ld_w_fd : desc->ld_w_df;
          st = mecefo_projection_refresh(desc->dtype, W[i], m, n, ldw, left ? 1 : 0, P[i].P, P[i].ld, P[i].r,
                                         policy->power_iters, policy->cond_steps, policy->polish_steps,
                                         const_cast<void*>(P[i].P), P[i].ld, ws, ws_bytes, hip_stream);
          if (st != MECEFO_OK) return st;
        }
      }
      st = mecefo_block_bwd_skip(desc, x.H, g, x.g_ffn, x.Wg, x.Wu, x.Wd, q.Pg, q.Pu, q.Pd, side, dX_bottom,
                                 q.dg_ffn, q.dWg, q.dWu, q.dWd, accumulate, ws, ws_bytes, hip_stream);
      if (st == MECEFO_OK && t) t[l] += 1;            // Alg. 3: the local step counter of this layer
    }
    if (st != MECEFO_OK) return st;
    g = dX_bottom;
  }
  return MECEFO_OK;
}

}  // extern "C"
