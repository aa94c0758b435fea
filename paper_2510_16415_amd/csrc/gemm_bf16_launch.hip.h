// Host-side launch helpers for the bf16 MFMA GEMM instantiations.
#pragma once
#include <float.h>
#include <math.h>

#include "gemm_bf16_dtl.hip.h"

namespace mecefo {

using CfgL4 = TileCfg<256, 256, 2, 2>;   // register staging, which only the "tile" option reaches
using CfgL8 = TileCfg<256, 256, 4, 2>;   // 8 waves x (64 x 128): two waves per SIMD hide latency
using CfgM = TileCfg<128, 128, 2, 2>;    // 4 waves x (64 x 64): two workgroups per CU
using CfgM8 = TileCfg<128, 128, 4, 2>;   // 8 waves x (32 x 64): one workgroup per CU
using CfgT = TileCfg<64, 64, 2, 2>;      // 4 waves x (32 x 32): three workgroups per CU
using CfgX = TileCfg<32, 32, 1, 1>;      // one wave, of eight that share out K
using CfgH = TileCfg<128, 256, 2, 4>;    // 8 waves x (64 x 64): half a large tile, in the last round of a launch
using CfgK = TileCfg<192, 256, 2, 4>;    // 8 waves x (96 x 64): three quarters of one

inline int cdiv(int a, int b) { return (a + b - 1) / b; }
constexpr int kMaxSplits = 16;   // parts a product may be cut into along K

// Two 64 KiB stages, refilled one stage ahead.  Measured alternatives that lost: four 32-K stages
// (64-byte row pieces double the L2 request count); rings of three buffers, symmetric or A2+B3 /
// A3+B2; a second barrier that lets two fills overlap; one operand staged through registers two
// stages ahead; line-touch prefetch of later stages (+8 %).  Fill latency is not what bounds the
// loop (a fills-only loop runs a stage in 0.9-1.3 us, the full loop gives it 1.4): LDS traffic of
// fills plus fragment reads and MFMA issue are both near a stage's length.  The power limit comes on top: the 7B-shaped
// layer takes 7 % longer on Gaussian than on all-zero operands.
using PipeL = DtlPipe<CfgL8, 2>;
// 64 KiB: two workgroups per CU cover each other's waits.  Four waves of 64 x 64 against eight of 32 x 64 (fewer LDS bytes
// per multiply-add, fewer waves to cover latency): a draw.  Calls with four waves, on two cards: [4096 x 1024] skip
// backward of two micro-batches 0.3 % slower and 1.5 % faster, [2048 x 2048] skip 1.8 and 1.1 % slower, 8-layer stack
// of [2048 x 512] 2.4 % slower on both, [4096 x 1024] forward equal and 1.4 % faster; mean of 16 and of 23 cases
// 0.6 and 0.3 % slower.
using PipeM2 = DtlPipe<CfgM, 2>;
using PipeM4 = DtlPipe<CfgM8, 4>;   // 128 KiB: one workgroup per CU, three stages in flight
using PipeH = DtlPipe<CfgH, 3>;    // 144 KiB
using PipeK = DtlPipe<CfgK, 2>;    // 112 KiB
using PipeT = DtlPipe<CfgT, 3>;    // 48 KiB
using PipeT2 = DtlPipe<CfgT, 3, 2>;   // 96 KiB: one workgroup per CU, two groups of waves share out K

using PipeX = DtlPipe<CfgX, 2, 8>;    // 128 KiB: eight groups of one wave

// ---- choice of the tile ------------------------------------------------------------------------
// What bounds a launch depends on how many workgroups it gives a CU.  One 256 x 256 workgroup per CU has
// the best rate (fewest operand bytes per multiply-add), but a K stage takes it 1.4 to 1.8 us however few
// of them there are, so a launch that fills a quarter of the chip pays the full length of K at that pace:
// smaller tiles walk K two to four times faster and give the idle CUs work.  The choice is the smallest
// modelled time over the configurations,
//     fixed + per_round * n + stages * max(stage_alone, stage_shared * n),   n = workgroups per CU
// (stage_alone .. stage_full between 96 and 256 workgroups on a CU each),
// with constants fitted to a sweep of 50 launches over every operand layout (K 32 to 11008, 2 to 2752
// workgroups; the model is within 15 % of nearly all of them).  Every launch of the sweep had one K; problems of
// different length are laid out over the CUs, the longest first.  Sides measured, in us (256^2 / 128^2
// two-stage / 128^2 four-stage / 64^2): [2048 x 2048], K 2048: 49 / 27 / 27 / 35; the same three in one
// launch: 54 / 60 / 73 / 84; [512 x 512], K 2048: 47 / 23 / 25 / 15; [2048 x 2048], K 5461: 135 / 80 / 61 /
// 101; [2048 x 512], K 1376: 33 / 16 / 17 / 11; SwiGLU recompute of 2048 tokens, d 2048, f 5461: 119 / 111 /
// 138 / 156; [4096 x 4096], K 8192: 248 / 310 / 383 / 456.  The register-staged 128 x 128 kernel that the
// small launches ran on before took 51, 81, 51, 99, 23, 143 and 624 us.
// The 64 x 64 workgroup is a chain of short stages (LDS reads, four MFMAs, barrier, fill addresses: 0.35 to 0.44 us);
// two groups of waves halve it where the CU would hold no second workgroup and K has sixteen stages to share:
// [2048 x 512], two segments of K 1376: 20.3 -> 16.5 us, [512 x 512], K 2048: 15.1 -> 12.0, K 512: 6.8 both.
// Launches of fewer 64 x 64 tiles than a quarter of the CUs take 32 x 32 ones: eight waves share out K, each fills and
// reads LDS buffers of its own and meets the others only to add up the tile, so that a CU has 64 to 128 KiB in flight
// and no barrier to wait at.  64 x 64 with two groups against 32 x 32, us: [512 x 512], K 512: 5.0 / 4.3, K 2048:
// 10.6 / 7.6, K 5461: 23.3 / 15.3; [129 x 200], K 512: 5.1 / 4.1; but [2048 x 512], K 512: 5.3 / 12.7 (1024 workgroups).
enum TileConfig : int { TILE_L = 0, TILE_M2 = 1, TILE_M4 = 2, TILE_T = 3, TILE_T2 = 4, TILE_K = 5, TILE_X = 6, TILE_COUNT = 7,
                        TILE_R4 = 7, TILE_R8 = 8,      // register-staged with four or eight waves: forced only
                        TILE_LT = 9 };                 // forced: TILE_L with its last round cut up where it can be

// No bound on the workgroups that share a CU: the rates of larger n are those of the fullest CU measured.
struct TileModel { int bm, bn; float fixed, per_round, stage_alone, stage_full, stage_shared; };
inline const TileModel& tile_model(int c) {
  static const TileModel m[TILE_COUNT] = {{256, 256, 3.5f, 2.5f, 1.45f, 1.75f, 1.75f},
                                          {128, 128, 2.0f, 1.0f, 0.86f, 0.86f, 0.62f},
                                          {128, 128, 2.6f, 0.9f, 0.69f, 0.69f, 0.72f},
                                          {64, 64, 2.0f, 0.5f, 0.33f, 0.36f, 0.28f},
                                          {64, 64, 2.6f, 0.5f, 0.23f, 0.26f, 0.45f},
                                          {192, 256, 3.5f, 2.2f, 1.20f, 1.45f, 1.47f},
                                          {32, 32, 2.4f, 0.9f, 0.10f, 0.15f, 0.15f}};
  return m[c];
}

// What the 192-row tile and the cut-up last round are built for: operands whose rows can be cut anywhere, and the
// epilogues of launches that can be large.
constexpr bool has_tile_k(bool akc, bool bkc, int epi) {
  return akc && (epi == EPI_STORE || (bkc && (epi == EPI_GRAD || epi == EPI_SWIGLU_FWD || epi == EPI_SWIGLU_BWD || epi == EPI_RESID)));
}
constexpr bool has_tile_x(int epi) { return epi != EPI_ATTN_P && epi != EPI_ATTN_DS && epi != EPI_ROPE; }
constexpr bool has_tail(bool akc, bool bkc, int epi) {
  return has_tile_k(akc, bkc, epi) || (!akc && !bkc && (epi == EPI_GRAD || epi == EPI_STORE));
}

// K stages of a workgroup of problem i, and the workgroups of the problem on bm x bn tiles.
inline int bf16_parts(const GemmProblem& p) { return p.splits > 1 ? p.splits : 1; }
inline int bf16_stages(const GemmLaunch& g, int i) {
  const GemmProblem& p = g.p[i];
  return cdiv(cdiv(p.K, kBK) * (p.nseg > 1 && !epi_is_dual(g.epi) ? p.nseg : 1), bf16_parts(p));
}
inline int bf16_units(const GemmLaunch& g, int i, int bm, int bn) {
  const GemmProblem& p = g.p[i];
  return cdiv(p.M, bm) * cdiv(p.N, epi_is_dual(g.epi) ? bn / 2 : bn) * (p.batch > 1 ? p.batch : 1) * bf16_parts(p);
}

// A K that is no multiple of 8 and not padded with zeros behind a K-contiguous operand.
inline bool bf16_ragged(const GemmLaunch& g) {
  for (int i = 0; i < g.nprob; ++i)
    if ((g.a_kcontig || g.b_kcontig) && (g.p[i].K % 8) && !g.p[i].kpad_ok) return true;
  return false;
}

// Whether the launch may go out on the 192-row tile.  Not a causal product whose contraction ends at the diagonal: its first
// operand (probabilities, dS) is written up to the end of the 256-block of the diagonal, and a tile with rows of two such
// blocks would read on, behind that, for the rows of the first.
inline bool bf16_takes_k(const GemmLaunch& g, bool ragged) {
  return has_tile_k(g.a_kcontig, g.b_kcontig, g.epi) && !ragged && g.p[0].causal != CAUSAL_K_UPTO_M;
}

// The last round of a launch on 256 x 256 tiles, when it holds at most 128 of them: each takes a CU the length of K at
// 1.75 us a stage while half the chip and more is idle.  Cut into halves, quarters or sixteenths the same tiles go to all
// CUs, which walk K at 1.0, 0.72 or 0.45 us a stage; whatever takes the least time, `saved` us less than the whole ones.
// Gradients with a short K are paced by their stores: there the rounds run into each other, the last one costs less than
// its length and the kernel that cuts it up 1 to 3 us a round.  Whole / cut up, us, fp32 gradients: expansions of 528 tiles
// and 8 stages 66.6 / 62.7, 612 and 8: 79 / 86, 600 and 16: 109 / 114, 1152 and 2: 77 / 92, 2064 and 16: 296 / 318; exact
// gradients of 360 and 16: 71 / 68, 288 and 24: 92 / 76, 1920 and 4: 147 / 156; bf16 ones: 528 and 8: 61.5 / 52,
// 1152 and 4: 79 / 85, 336 and 16: 61 / 57.  So below 24 stages only with one or two full rounds, and only where what is saved is more than
// that.  (forced: wherever it is shorter by the stages alone.)
struct TailPlan { int tiles, shift, prob; float saved; };
inline TailPlan bf16_tail(const GemmLaunch& g, bool forced = false) {
  TailPlan plan = {0, 0, 0, 0.f};
  if (!has_tail(g.a_kcontig, g.b_kcontig, g.epi) || bf16_ragged(g)) return plan;
  int total = 0, most = 0;
  for (int i = 0; i < g.nprob; ++i) {
    const GemmProblem& p = g.p[i];
    if (p.batch > 1 || p.splits > 1 || (p.nseg > 1 && !epi_is_dual(g.epi)) || p.causal != CAUSAL_NONE || bf16_stages(g, i) != bf16_stages(g, 0)) return plan;
    const int u = bf16_units(g, i, 256, 256);
    total += u;
    if (u > most) { most = u; plan.prob = i; }
  }
  const int rest = total % kCUs;
  if (total < kCUs || rest == 0 || rest > kCUs / 2 || rest >= most || total >= 1 << 24) return plan;
  const float st = (float)bf16_stages(g, 0), rate[3] = {1.0f, 0.72f, 0.45f};
  const int shift[3] = {1, 2, 4}, rounds = total / kCUs;
  float lost = 0.f;
  if (g.epi == EPI_GRAD && st < 24.f && !forced) {
    if (rounds > 2) return plan;
    lost = g.out_f32 ? 4.f + 0.08f * rest + 1.2f * rounds : 2.f + 0.03f * rest + 0.5f * rounds;
  }
  for (int k = 0; k < 3; ++k) {
    const float saved = 4.f + 1.75f * st - lost - cdiv(rest << shift[k], kCUs) * (4.f + rate[k] * st);
    if (saved > plan.saved) { plan.saved = saved; plan.shift = shift[k]; plan.tiles = rest; }
  }
  return plan;
}

// The K stages of a launch's workgroups, the same on every configuration.
struct Stages {
  int of[kMaxProblems], longest = 0;
  bool equal = true;
  explicit Stages(const GemmLaunch& g) {
    for (int i = 0; i < g.nprob; ++i) {
      of[i] = bf16_stages(g, i);
      longest = of[i] > longest ? of[i] : longest;
      equal &= of[i] == of[0];
    }
  }
};

// Modelled time in us of the launch on configuration c.  Where it is seen early that this is not below `bound`, some value
// that is not below it either: laying out problems of different length takes 0.1 to 0.4 us, most of the planning of a launch.
inline float bf16_tile_cost(const GemmLaunch& g, int c, const Stages& st, float bound) {
  const TileModel& m = tile_model(c);
  const int* stages = st.of;
  const int longest = st.longest;
  const bool equal = st.equal;
  int units[kMaxProblems], total = 0;
  int64_t sum = 0;
  for (int i = 0; i < g.nprob; ++i) {
    units[i] = bf16_units(g, i, m.bm, m.bn);
    total += units[i];
    sum += (int64_t)units[i] * stages[i];
  }
  // up to a workgroup per CU: a stage takes longer the more of them there are (256 x 256: 1.45 us up to 96, 1.65 with 176)
  const float full = fminf(fmaxf((total - 96) / 160.f, 0.f), 1.f);
  const float alone = m.stage_alone + full * (m.stage_full - m.stage_alone);
  float n = total / 256.f, load;               // workgroups and K stages of the fullest CU
  const bool few = n < 4.f;                    // workgroups per CU: the fullest CU sets the time
  if (equal || !few) {
    // the 192-row tile's last round counts in full behind more of them as well, and is never cut up: 1045 such tiles with 64
    // stages take 478 us, five rounds of 95, where 4.1 would be 390
    if (few || c == TILE_K) n = (float)(int)(n + 0.999f);
    load = 0.f;
    for (int i = 0; i < g.nprob; ++i) load += (float)units[i] * stages[i];
    load *= n / total;
  } else {
    const float least = fmaxf((float)longest, sum / 256.f);   // the fullest CU holds the longest problem's stages, and the mean
    const float t = m.fixed + m.per_round + (total <= kCUs ? least * alone : fmaxf(longest * m.stage_alone, least * m.stage_shared));
    if (t >= bound * 1.0001f) return t;
    // Problems of different length, the longest first, each workgroup to the CU with the least to do.  At most
    // 2 * kMaxProblems * 4 groups of equally loaded CUs come about: a problem fills whole groups, and splits one.
    struct { int load, cus, wgs; } q[64] = {{0, 256, 0}};
    int nq = 1;
    bool done[kMaxProblems] = {};
    for (int k = 0; k < g.nprob; ++k) {
      int i = -1;
      for (int j = 0; j < g.nprob; ++j)
        if (!done[j] && (i < 0 || stages[j] > stages[i])) i = j;
      done[i] = true;
      for (int left = units[i]; left > 0 && nq < 64;) {
        int at = 0;
        for (int j = 1; j < nq; ++j)
          if (q[j].load < q[at].load) at = j;
        const int take = left < q[at].cus ? left : q[at].cus;
        if (take < q[at].cus) {
          q[nq] = q[at];
          q[nq++].cus -= take;
          q[at].cus = take;
        }
        q[at].load += stages[i];
        q[at].wgs += 1;
        left -= take;
      }
    }
    int at = 0;
    for (int j = 1; j < nq; ++j)
      if (q[j].load > q[at].load) at = j;
    load = (float)q[at].load;
    n = (float)q[at].wgs;
  }
  const float time = total <= kCUs ? load * alone : fmaxf(longest * m.stage_alone, load * m.stage_shared);
  return m.fixed + m.per_round * n + time - (c == TILE_L && few && equal ? bf16_tail(g).saved : 0.f);
}
inline float bf16_tile_cost(const GemmLaunch& g, int c) { return bf16_tile_cost(g, c, Stages(g), FLT_MAX); }

// The configuration of the smallest modelled time; with a `bound`, only if that is below it.
inline int bf16_best_tile(const GemmLaunch& g, float* cost = nullptr, float bound = FLT_MAX) {
  const Stages st(g);
  const bool ragged = bf16_ragged(g);
  int best = TILE_L;
  float t = bound;
  for (int c = 0; c < TILE_COUNT; ++c) {
    if (c == TILE_X && !has_tile_x(g.epi)) continue;
    if (c == TILE_K && !bf16_takes_k(g, ragged)) continue;
    // with a ragged K the groups of waves meet one more barrier per stage: a third of what they save
    const float x = bf16_tile_cost(g, c, st, t) + (c == TILE_T2 && ragged ? 0.05f * st.longest : 0.f);
    if (x < t) { t = x; best = c; }
  }
  if (cost) *cost = t;
  return best;
}

// Cuts the problems of a store launch along K (their `splits`) where that makes the launch shorter, into parts of about
// equal length with four or more stages each, of which `room` fp32 elements can be held (parts_room for read_parts).  The parts are written, read
// back and summed by one more launch: 4 us and their bytes, at about 5 TB/s each way while the cache behind the L2s holds
// them (the sum of 59 MB takes 11 us, of 4 MB 5 us), at 3 beyond; parts that their reader adds up itself cost their bytes.  Returns the modelled time of it all.
inline float bf16_plan_splits(GemmLaunch& g, int64_t room, int64_t parts_room = 0) {
  int longest = 0;
  for (int i = 0; i < g.nprob; ++i) {
    g.p[i].splits = 1;
    longest = bf16_stages(g, i) > longest ? bf16_stages(g, i) : longest;
  }
  float t;
  bf16_best_tile(g, &t);
  int best[kMaxProblems];
  for (int i = 0; i < g.nprob; ++i) best[i] = 1;
  for (int s = 2; s <= kMaxSplits && longest / s >= 4; ++s) {
    const int len = cdiv(longest, s);
    int64_t out = 0, read = 0;
    for (int i = 0; i < g.nprob; ++i) {
      g.p[i].splits = 1;
      const int whole = bf16_stages(g, i);
      int parts = !g.p[i].whole && whole > len + len / 8 ? cdiv(whole, len) : 1;
      if (g.p[i].read_parts && parts > kMaxNormParts) parts = kMaxNormParts;
      g.p[i].splits = parts;
      if (parts > 1) (g.p[i].read_parts ? read : out) += (int64_t)parts * g.p[i].M * g.p[i].ldc;
    }
    const float extra = (out > 0 ? 4.f : 0.f) + (float)out * (out < 32 << 20 ? 1.0e-6f : 2.7e-6f) +
                        (float)read * (read < 32 << 20 ? 0.6e-6f : 2.0e-6f);
    if (out > room || read > parts_room || extra >= t) break;   // more parts are more bytes
    float x;
    const float bound = t - extra;
    bf16_best_tile(g, &x, bound);
    if (x < bound) {
      t = x + extra;
      for (int i = 0; i < g.nprob; ++i) best[i] = g.p[i].splits;
    }
  }
  for (int i = 0; i < g.nprob; ++i) g.p[i].splits = best[i];
  return t;
}

struct NoPipe { static constexpr int LDS_BYTES = 0, THREADS = 0; };

// One kernel instantiation: its entry point, its dynamic LDS size and the once-per-device limit raise.
template <class Cfg, bool AKC, bool BKC, int EPI, class Pipe, bool RAGGED>
struct Bf16Kernel {
  static constexpr bool DTL = Pipe::LDS_BYTES > 0;
  static constexpr int LDS = DTL ? Pipe::LDS_BYTES : Cfg::LDS_BYTES;
  static auto entry() -> void (*)(const KArgs) {
    if constexpr (DTL) return gemm_bf16_dtl_kernel<Cfg, Pipe, AKC, BKC, EPI, RAGGED>;
    else return gemm_bf16_kernel<Cfg, AKC, BKC, EPI>;
  }
  static hipError_t prepare() {
    static LdsLimitOnce limit;
    return limit.ensure((const void*)entry(), LDS);
  }
};

template <class Cfg, bool AKC, bool BKC, int EPI, class Pipe = NoPipe, bool RAGGED = true>
hipError_t run_bf16(GemmLaunch& g, hipStream_t stream) {
  using Kern = Bf16Kernel<Cfg, AKC, BKC, EPI, Pipe, RAGGED>;
  constexpr int LDS = Kern::LDS;
  constexpr bool DUAL = epi_is_dual(EPI);
  KArgs a;
  fill_kargs(a, g, Cfg::BM, DUAL ? Cfg::BN / 2 : Cfg::BN, kBK);
  if (a.h.total == 0) return hipSuccess;
  const hipError_t e = Kern::prepare();
  if (e != hipSuccess) return e;
  const unsigned side = add_side(a, g, Kern::DTL ? side_kind(AKC, BKC, EPI) : SIDE_NONE, Pipe::THREADS);
  hipLaunchKernelGGL(Kern::entry(), dim3(a.h.total + side), dim3(Kern::DTL ? Pipe::THREADS : Cfg::NT), LDS, stream, a);
  return hipGetLastError();
}

// The launch whose last round is cut up as `plan` says.
template <bool AKC, bool BKC, int EPI>
struct TailKernel {
  static constexpr int LDS = PipeH::LDS_BYTES;
  static_assert(LDS >= PipeL::LDS_BYTES && LDS >= PipeM4::LDS_BYTES && LDS >= PipeT2::LDS_BYTES, "the largest of them");
  static auto entry() -> void (*)(const KArgs) {
    return gemm_bf16_tail_kernel<CfgL8, PipeL, CfgH, PipeH, CfgM8, PipeM4, CfgT, PipeT2, AKC, BKC, EPI>;
  }
  static hipError_t prepare() {
    static LdsLimitOnce limit;
    return limit.ensure((const void*)entry(), LDS);
  }
};
template <bool AKC, bool BKC, int EPI>
hipError_t run_bf16_tail(GemmLaunch& g, const TailPlan& plan, hipStream_t stream) {
  using Kern = TailKernel<AKC, BKC, EPI>;
  KArgs a;
  fill_kargs(a, g, CfgL8::BM, epi_is_dual(EPI) ? CfgL8::BN / 2 : CfgL8::BN, kBK);
  for (int s = 0; s < kMaxProblems; ++s)
    if ((a.h.order >> (4 * s) & 15) == plan.prob) {
      a.h.units[s] -= plan.tiles;
      a.h.total -= plan.tiles;
      a.h.tail = plan.prob << 28 | plan.shift << 24 | a.h.units[s];
      break;
    }
  const hipError_t e = Kern::prepare();
  if (e != hipSuccess) return e;
  a.h.gemm_blocks = a.h.total + (plan.tiles << plan.shift);
  const unsigned side = add_side(a, g, side_kind(AKC, BKC, EPI), PipeL::THREADS);
  hipLaunchKernelGGL(Kern::entry(), dim3(a.h.gemm_blocks + side), dim3(PipeL::THREADS), Kern::LDS, stream, a);
  return hipGetLastError();
}

// The register-staged kernels serve as a second implementation in tests only; the epilogues of the projection refresh,
// the residual adds and the rotation are not built for them, and such launches take the 256 x 256 direct-to-LDS tile
// where a register-staged one is forced.
constexpr bool register_staged(int epi) { return epi != EPI_POLY && epi != EPI_HILO && epi != EPI_RESID && epi != EPI_ROPE; }

// Limit raise for the configurations of one (layout, epilogue) pair.
template <bool AKC, bool BKC, int EPI>
hipError_t prepare_bf16() {
  hipError_t e = Bf16Kernel<CfgL8, AKC, BKC, EPI, PipeL, false>::prepare();
  if (e == hipSuccess && (AKC || BKC)) e = Bf16Kernel<CfgL8, AKC, BKC, EPI, PipeL, AKC || BKC>::prepare();
  if (e == hipSuccess) e = Bf16Kernel<CfgM, AKC, BKC, EPI, PipeM2, true>::prepare();
  if (e == hipSuccess) e = Bf16Kernel<CfgM8, AKC, BKC, EPI, PipeM4, true>::prepare();
  if (e == hipSuccess) e = Bf16Kernel<CfgT, AKC, BKC, EPI, PipeT, true>::prepare();
  if (e == hipSuccess) e = Bf16Kernel<CfgT, AKC, BKC, EPI, PipeT2, true>::prepare();
  if constexpr (has_tile_x(EPI)) {
    if (e == hipSuccess) e = Bf16Kernel<CfgX, AKC, BKC, EPI, PipeX, true>::prepare();
  }
  if constexpr (has_tile_k(AKC, BKC, EPI)) {
    if (e == hipSuccess) e = Bf16Kernel<CfgK, AKC, BKC, EPI, PipeK, false>::prepare();
  }
  if constexpr (has_tail(AKC, BKC, EPI)) {
    if (e == hipSuccess) e = TailKernel<AKC, BKC, EPI>::prepare();
  }
  if constexpr (register_staged(EPI)) {
    if (e == hipSuccess) e = Bf16Kernel<CfgL4, AKC, BKC, EPI, NoPipe, true>::prepare();
    if (e == hipSuccess) e = Bf16Kernel<CfgL8, AKC, BKC, EPI, NoPipe, true>::prepare();
  }
  return e;
}

// The configuration mecefo_set_option("tile", ...) forces, -1 when the model decides.  Another host thread may change
// the option at any time: whoever needs the answer twice for one launch keeps it.
inline int bf16_forced_tile() {
  static const int tile[kTileOptions] = {-1, TILE_M2, TILE_R4, TILE_R8, TILE_L, TILE_M4, TILE_T, TILE_T2, TILE_K, TILE_LT, TILE_X};
  return tile[options().tile.load(std::memory_order_relaxed)];
}

template <bool AKC, bool BKC, int EPI>
hipError_t run_bf16_auto(GemmLaunch& g, hipStream_t stream) {
  const int forced = bf16_forced_tile(), c = forced < 0 ? bf16_best_tile(g) : forced;
  if constexpr (register_staged(EPI)) {
    if (c == TILE_R4) return run_bf16<CfgL4, AKC, BKC, EPI>(g, stream);
    if (c == TILE_R8) return run_bf16<CfgL8, AKC, BKC, EPI>(g, stream);
  }
  switch (c) {
    case TILE_M2: return run_bf16<CfgM, AKC, BKC, EPI, PipeM2>(g, stream);
    case TILE_M4: return run_bf16<CfgM8, AKC, BKC, EPI, PipeM4>(g, stream);
    case TILE_T: return run_bf16<CfgT, AKC, BKC, EPI, PipeT>(g, stream);
    case TILE_T2: return run_bf16<CfgT, AKC, BKC, EPI, PipeT2>(g, stream);
    default:
      if constexpr (has_tile_x(EPI)) {
        if (c == TILE_X) return run_bf16<CfgX, AKC, BKC, EPI, PipeX>(g, stream);
      }
      if constexpr (has_tile_k(AKC, BKC, EPI)) {
        if (c == TILE_K && bf16_takes_k(g, bf16_ragged(g))) return run_bf16<CfgK, AKC, BKC, EPI, PipeK, false>(g, stream);
      }
      if constexpr (has_tail(AKC, BKC, EPI)) {
        const TailPlan plan = bf16_tail(g, forced == TILE_LT);
        if (plan.saved > 0.f && (forced < 0 || forced == TILE_LT)) return run_bf16_tail<AKC, BKC, EPI>(g, plan, stream);
      }
      if (bf16_ragged(g)) return run_bf16<CfgL8, AKC, BKC, EPI, PipeL, AKC || BKC>(g, stream);
      return run_bf16<CfgL8, AKC, BKC, EPI, PipeL, false>(g, stream);
  }
}

hipError_t launch_gemm_bf16_nt(GemmLaunch& g, hipStream_t s);
hipError_t launch_gemm_bf16_nn(GemmLaunch& g, hipStream_t s);
hipError_t launch_gemm_bf16_tn(GemmLaunch& g, hipStream_t s);

}  // namespace mecefo
