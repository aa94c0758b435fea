// bf16 MFMA GEMM for gfx950 with direct-to-LDS operand staging.
//
// One workgroup computes a tile of 256 x 256 (eight wavefronts of 64 x 128), 192 x 256 (eight of 96 x 64), 128 x 128 (four of
// 64 x 64 with two LDS stages, or eight of 32 x 64 with four), 64 x 64 (four of 32 x 32, or two groups of four that share
// out K) or 32 x 32 (eight waves that share out K, each with buffers of its own).  Two differences to
// gemm_bf16.hip.h.  The products run on v_mfma_f32_16x16x32_bf16: on Gaussian operands a loop of nothing but MFMAs is
// power-limited, and this shape moves half the accumulator bytes per multiply-add of the 32x32x16 one -- 2100 TFLOP/s
// at 2.1 GHz on random operands against 1860 at 1.83 GHz.  And the operand tiles never pass through registers:
// `buffer_load_dwordx4 ... lds` writes 1 KiB per wavefront instruction straight into LDS
// (lane i lands at base + 16 i).  K is cut into stages of BK (32 or 64) held in a ring of NS
// LDS buffers; a buffer is refilled as soon as the barrier that ends its last use has passed,
// NS - 1 stages ahead of its next use, and the kernel waits (vmcnt) only for the stage it is
// about to read, leaving the younger fills in flight.
//   * K-contiguous operands keep the XOR-swizzled [rows][64] layout: the swizzle is applied by
//     choosing which 16-byte chunk of the row each lane fetches.
//   * K-strided operands ([K x rows] in memory: weights used as [K x N], activations in the
//     token contraction) stay in their memory order [64 k][tile rows] in LDS and are transposed
//     on the way to the MFMA registers by ds_read_b64_tr_b16 (each 16-lane group turns four
//     k-rows of 16 elements into four K-consecutive values per lane); their 16-byte chunks are
//     XOR-swizzled by k so that the eight k-rows of a 32-lane pass fall into different banks.
// Rows and K positions outside the matrices are fetched from outside the buffer (zeros).
// A K-contiguous operand whose K ends inside a 16-byte chunk has that chunk cleaned in LDS after it has
// landed (clear_tail); the host says which problems need it.
#pragma once
#include "gemm_bf16.hip.h"

namespace mecefo {

typedef __attribute__((ext_vector_type(4))) short s16x4_t;

// Buffer resource as four scalar words: base address, stride 0, 2 GiB range, raw dword format.
__device__ inline u32x4_t make_rsrc_words(const void* p) {
  const uint64_t a = (uint64_t)p;
  u32x4_t r;
  r[0] = (uint32_t)a;
  r[1] = (uint32_t)(a >> 32) & 0xFFFFu;
  r[2] = 0x7FFFFFFFu;
  r[3] = 0x00020000u;
  return r;
}

// Wave-uniform choice between the descriptors of up to three K segments.  Only the base words
// differ; they are selected word by word and pinned to scalar registers (a vector-typed select is
// otherwise lowered to vector moves, which the fill instruction cannot take).
__device__ inline u32x4_t select_rsrc(int seg, const u32x4_t& r0, const u32x4_t& r1, const u32x4_t& r2) {
  u32x4_t r = r0;
  r[0] = __builtin_amdgcn_readfirstlane(seg == 0 ? r0[0] : (seg == 1 ? r1[0] : r2[0]));
  r[1] = __builtin_amdgcn_readfirstlane(seg == 0 ? r0[1] : (seg == 1 ? r1[1] : r2[1]));
  return r;
}

__device__ inline uint32_t lds_address(const void* p) {
  return (uint32_t)(size_t)(__attribute__((address_space(3))) const uint8_t*)p;
}

// One wavefront-wide fill: lane i fetches 16 bytes at voff + soff and they land at lds_addr + 16 i.
// Written as inline assembly so that the compiler does not serialise later LDS reads of the other
// stage behind it; the kernel waits for these loads itself (wait_fills) before the stage barrier.
__device__ inline void fill_lds_16B(u32x4_t rsrc, uint32_t lds_addr, uint32_t voff, uint32_t soff) {
  asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
               :: "s"(lds_addr), "v"(voff), "s"(rsrc), "s"(soff) : "memory");
}
// Wait until at most `stages_left` younger stages (FPS fill instructions each, per wave) are in flight.
template <int FPS>
__device__ inline void wait_fills_leave(int stages_left) {
  if (stages_left <= 0) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(0) : "memory");
  else if (stages_left == 1) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(FPS) : "memory");
  else if (stages_left == 2) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(2 * FPS) : "memory");
  else if (stages_left == 3) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(3 * FPS) : "memory");
  else if (stages_left == 4) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(4 * FPS) : "memory");
  else asm volatile("s_waitcnt vmcnt(%0)" :: "n"(5 * FPS) : "memory");
}

// ---- direct-to-LDS fill of one operand tile (ROWS rows x BK) -------------------------------
// Swizzle of the K-contiguous layout [rows][BK]: physical 16-byte chunk = logical ^ kc_swz(row).
// A 16-byte read of the 16x16x32 operand (lane l: row l % 16, chunk l / 16 of the step) is served 16
// lanes per clock, and the lanes of a clock are eight rows at one chunk plus the other eight rows of
// the block at the neighbouring chunk (lanes 0-7 with 24-31, 8-15 with 16-23, and the same in the
// upper half-wave; found by measurement: SQ_LDS_BANK_CONFLICT).  Rows of equal parity share their half
// of the 64 banks; XORing row bits 1-2 into chunk bits 1-2 spreads the four rows of a parity over the
// even (or odd) chunks and leaves the other chunks to the neighbouring-chunk rows.
template <int BK> __device__ inline int kc_swz(int row) {
  if constexpr (BK == 64) return row & 6;                  // 8 chunks per 128-byte row
  else return ((row >> 1) ^ (row >> 3)) & 3;               // 4 chunks per 64-byte row
}

template <int BK, int NT, int ROWS, bool DUAL>
struct DmaKC {   // K-contiguous source; one wave instruction covers RPI consecutive rows
  static constexpr int ROWB = BK * 2, CH = ROWB / 16, RPI = 1024 / ROWB;
  static constexpr int NW = NT / 64, NI = (ROWS / RPI) / NW;
  static_assert(NI >= 1 && (!DUAL || NI % 2 == 0), "unsupported stage size");
  uint32_t voff[NI];
  int c;       // logical 16-byte chunk this lane fetches (the same for all its instructions)
  int w;
  __device__ inline void init(int lane, int wave, int row_base, int rows_total, int64_t ld) {
    w = wave;
    const int rsub = lane / CH;
    c = (lane % CH) ^ kc_swz<BK>(w * RPI + rsub);   // instructions q*NW + w differ by multiples of NW * RPI rows
#pragma unroll
    for (int q = 0; q < NI; ++q) {
      const int row = (q * NW + w) * RPI + rsub;
      const int gr = row_base + (DUAL ? (row & (ROWS / 2 - 1)) : row);
      voff[q] = gr < rows_total ? ((uint32_t)gr * (uint32_t)ld + c * 8) * 2 : kOOB;      // operands lie below 2 GiB
    }
  }
  __device__ inline void issue(u32x4_t r0, u32x4_t r1, uint32_t tile, int k0, int K, bool tail) const {
    const bool kvalid = !tail || (k0 + c * 8 < K);
#pragma unroll
    for (int q = 0; q < NI; ++q) {
      const uint32_t off = kvalid ? voff[q] : kOOB;
      fill_lds_16B((DUAL && q >= NI / 2) ? r1 : r0, tile + (q * NW + w) * 1024, off, (uint32_t)k0 * 2);
    }
  }
  // A ragged K ends inside a 16-byte chunk, whose rest holds bytes from behind the rows: zero the last
  // 8 - rem elements of that chunk (index kend / 8 of the stage, rem = kend % 8) in every row of a landed tile.
  static __device__ inline void clear_tail(uint8_t* tile, int t, int kend) {
    for (int row = t; row < ROWS; row += NT) {
      __bf16* chunk = (__bf16*)(tile + row * ROWB + (((kend >> 3) ^ kc_swz<BK>(row)) << 4));
      for (int e = kend & 7; e < 8; ++e) chunk[e] = (__bf16)0.f;
    }
  }
};

// Physical 16-byte chunk of logical chunk c (eight columns each) in k row k of a K-strided tile
// [BK k][ROWS], and back.  A transposing read takes, per pass of 32 lanes, 32 bytes (two chunks) of each
// of eight k rows: four consecutive ones and the four that lie eight further on (the two 16-lane groups of
// a pass hold neighbouring K groups of the 16x16x32 operand).  LDS serves 256 bytes per clock from 64
// banks, so the 16 chunks of a pass must fall on different sixteenths of 256 bytes.  Rows of 256 or 512
// bytes: bit 0 is the chunk of the pair, the k row fills bits 1-2 (XOR with its low bits) and bit 3 (XOR
// with k bits 2 and 3); the second chunk pair of a row (bit 1 of c) also goes to the other half of the
// banks.  Rows of 128 bytes: k bit 0 is the half of the banks by itself, k bits 1 and 3 fill chunk bits 1-2.
// The map is its own inverse.
template <int ROWS> struct KsMap {
  static constexpr int CH = ROWS / 8;
  static_assert(ROWS == 32 || ROWS == 64 || ROWS == 128 || ROWS == 256, "unsupported tile width");
  static __device__ inline int fold(int c) { return ROWS <= 64 ? c : c ^ ((c & 2) << 2); }
  static __device__ inline int swz(int k) {
    return ROWS == 32 ? (k & 8) >> 2 : ROWS == 64 ? (k & 2) | ((k & 8) >> 1) : ((k & 7) << 1) ^ (k & 8);
  }
  static __device__ inline int phys(int c, int k) { return (fold(c) ^ swz(k)) & (CH - 1); }
  static __device__ inline int logical(int pos, int k) { return fold((pos ^ swz(k)) & (CH - 1)); }
};

template <int BK, int NT, int ROWS>
struct DmaKS {   // K-strided source; one wave instruction covers KPI k rows of 2 * ROWS bytes
  static constexpr int ROWB = ROWS * 2, CH = ROWB / 16, KPI = 1024 / ROWB;
  static constexpr int NW = NT / 64, NI = (BK / KPI) / NW;
  // the swizzle sees k % 16: one lane offset for all instructions, or two that take turns
  static constexpr int NV = NI == 1 || (NW * KPI) % 16 == 0 ? 1 : 2;
  static_assert(NI >= 1 && (NV == 1 || (NW * KPI) % 16 == 8), "unsupported stage size");
  uint32_t voff[NV];  // lane offset of k row krow0; instruction q adds NW * KPI * q rows
  uint32_t ld2;
  int krow0;          // k row of this lane for q = 0
  int w;
  __device__ inline void init(int lane, int wave, int row_base, int rows_total, int64_t ld) {
    w = wave;
    krow0 = KPI * w + lane / CH;
    ld2 = (uint32_t)(ld * 2);
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const int m = row_base + KsMap<ROWS>::logical(lane % CH, krow0 + v * NW * KPI) * 8;
      voff[v] = m < rows_total ? ((uint32_t)krow0 * (uint32_t)ld + m) * 2 : kOOB;
    }
  }
  __device__ inline void issue(u32x4_t r0, u32x4_t, uint32_t tile, int k0, int K, bool tail) const {
    const uint32_t soff = (uint32_t)k0 * ld2;
#pragma unroll
    for (int q = 0; q < NI; ++q) {
      const bool kvalid = !tail || (k0 + krow0 + NW * KPI * q < K);
      const uint32_t v = voff[q % NV];
      const uint32_t off = (kvalid && v != kOOB) ? v + (uint32_t)(NW * KPI * q) * ld2 : kOOB;
      fill_lds_16B(r0, tile + (q * NW + w) * 1024, off, soff);
    }
  }
  static __device__ inline void clear_tail(uint8_t*, int, int) {}   // whole k rows are masked by the fills
};

template <int BK, int NT, int ROWS, bool KC, bool DUAL> struct DmaSel { using type = DmaKC<BK, NT, ROWS, DUAL>; };
template <int BK, int NT, int ROWS, bool DUAL> struct DmaSel<BK, NT, ROWS, false, DUAL> {
  static_assert(!DUAL, "dual products need K-contiguous B");
  using type = DmaKS<BK, NT, ROWS>;
};

// ---- MFMA operand fetch from LDS ------------------------------------------------------
// Operands of v_mfma_f32_16x16x32_bf16: NB blocks of 16 rows; lane l holds row l % 16 and the eight
// K values 8 (l / 16) .. + 7 of a 32-K step.  K-contiguous tiles: one ds_read_b128 per block and step.
template <int BK, int NB, int ROWS>
struct FragKC {
  int base[NB];
  // rows[i]: first tile row of block i for this wave
  __device__ inline void init(int lane, const int (&rows)[NB]) {
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int row = rows[i] + (lane & 15);
      base[i] = row * (BK * 2) + (((lane >> 4) ^ kc_swz<BK>(row)) << 4);
    }
  }
  __device__ inline bf16x8_t fetch_one(int i, const uint8_t* tile, int step) const {
    return *(const bf16x8_t*)(tile + (base[i] ^ (step << 6)));
  }
};

// K-strided tiles ([BK k][ROWS]): two transposing 8-byte reads per block.  Within
// a 16-lane group source lane 4 kq + q4 supplies rows 4 q4 .. + 3 at k row kq; the read hands result
// lane i the four K-consecutive values of row i.
template <int BK, int NB, int ROWS>
struct FragKS {
  static constexpr int ROWB = ROWS * 2;
  int base[NB][2];
  __device__ inline void init(int lane, const int (&rows)[NB]) {
    const int kq = (lane & 15) >> 2, g = lane >> 4, q4 = lane & 3;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int m = rows[i] + 4 * q4;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int k = 8 * g + 4 * h + kq;
        base[i][h] = k * ROWB + (KsMap<ROWS>::phys(m >> 3, k) << 4) + ((m & 7) << 1);
      }
    }
  }
  __device__ inline bf16x8_t fetch_one(int i, const uint8_t* tile, int step) const {
    typedef __attribute__((address_space(3))) s16x4_t lds_s16x4_t;
    const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)(tile + base[i][0] + step * 32 * ROWB));
    const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)(tile + base[i][1] + step * 32 * ROWB));
    typedef __attribute__((ext_vector_type(8))) short s16x8_t;
    const s16x8_t v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8_t, v);
  }
};

template <int BK, int NB, int ROWS, bool KC> struct FragSel { using type = FragKC<BK, NB, ROWS>; };
template <int BK, int NB, int ROWS> struct FragSel<BK, NB, ROWS, false> { using type = FragKS<BK, NB, ROWS>; };

// Pipeline shape of the direct-to-LDS kernel for a tile: 64 K elements per stage, KG groups of Cfg::NT threads
// that take the stages in turn (each with NS LDS buffers of its own) and add up their tiles at the end.
template <class Cfg, int NS_, int KG_ = 1> struct DtlPipe {
  static constexpr int BK = 64, NS = NS_, KG = KG_, THREADS = Cfg::NT * KG;
  static constexpr int A_BYTES = Cfg::BM * BK * 2, B_BYTES = Cfg::BN * BK * 2, STAGE_BYTES = A_BYTES + B_BYTES;
  static constexpr int NW = Cfg::NT / 64;
  static constexpr int FPS = STAGE_BYTES / 1024 / NW;      // fill instructions per wave and stage
  // per-wave LDS slice of the staged epilogue: 32 rows x (WN + 4) floats, or 2 x 32 x (WN / 2 + 4)
  static constexpr int EP_WAVE_BYTES = 32 * (Cfg::WN + 8) * 4;
  static constexpr int SUM_BYTES = (KG - 1) * Cfg::BM * Cfg::BN * 4;      // the other groups' tiles, behind the epilogue slices
  static constexpr int EP_BYTES = NW * EP_WAVE_BYTES + SUM_BYTES;
  static constexpr int LDS_BYTES = KG * NS * STAGE_BYTES > EP_BYTES ? KG * NS * STAGE_BYTES : EP_BYTES;
  static_assert(NS >= 2 && NS <= 4 && LDS_BYTES <= 160 * 1024 && (NS - 1) * FPS <= 63, "bad pipeline");
};

// RAGGED: K may end inside a 16-byte chunk (the instantiation without it keeps the large tile's loop free of the
// test: 0.5 % of the 7B-shaped layer).
// SEGS: products may have several K segments.
template <class Cfg, class Pipe, bool AKC, bool BKC, int EPI, bool RAGGED, bool SEGS>
__device__ __forceinline__ void dtl_tile(const KHead& head, GemmProblem p, int m0, int n0, int split, uint8_t* smem_all) {
  constexpr bool DUAL = epi_is_dual(EPI);
  constexpr int BM = Cfg::BM, BN = Cfg::BN, NT = Cfg::NT;
  constexpr int TM = Cfg::WM / 16, TN = Cfg::WN / 16;     // 16x16 MFMA blocks per wave
  constexpr int BK = Pipe::BK, NS = Pipe::NS, KS = BK / 32, FPS = Pipe::FPS;
  constexpr int A_BYTES = Pipe::A_BYTES, STAGE = Pipe::STAGE_BYTES, KG = Pipe::KG;
  static_assert(TM % 2 == 0 && TN % (DUAL ? 2 : 1) == 0, "the epilogue takes 32 rows at a time");
  const int group = KG > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / NT) : 0;
  const int t = threadIdx.x - group * NT;      // thread, wave and LDS buffers within the group
  const int lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  uint8_t* smem = smem_all + group * NS * STAGE;
  const int wm = wave / Cfg::WAVES_N, wn = wave % Cfg::WAVES_N;

  const int nseg = DUAL || !SEGS ? 1 : p.nseg;
  const int K = p.K;
  const int kt_per_seg = (uint32_t)(K + BK - 1) / BK;
  const int kt_total = kt_per_seg * nseg;
  int kt_begin = split * p.chunk;
  int kt_end = min(kt_total, kt_begin + p.chunk);
  causal_clip(p, m0, n0, BM, BK, kt_begin, kt_end);

  using DmaA = typename DmaSel<BK, NT, BM, AKC, false>::type;
  using DmaB = typename DmaSel<BK, NT, BN, BKC, DUAL>::type;
  DmaA da;
  DmaB db;
  da.init(lane, wave, m0, p.M, p.lda);
  db.init(lane, wave, n0, p.N, p.ldb);
  const u32x4_t ra0 = make_rsrc_words(p.A[0]);
  const u32x4_t ra1 = make_rsrc_words(p.A[1]);
  const u32x4_t rb0 = make_rsrc_words(p.B[0]);
  const u32x4_t rb1 = make_rsrc_words(p.B[1]);
  const u32x4_t ra2 = make_rsrc_words(p.A[2]);
  const u32x4_t rb2 = make_rsrc_words(p.B[2]);
  const uint32_t smem_addr = lds_address(smem);

  int a_rows[TM], b_rows[TN];
#pragma unroll
  for (int i = 0; i < TM; ++i) a_rows[i] = wm * Cfg::WM + i * 16;
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    if constexpr (DUAL) b_rows[j] = (j >= TN / 2 ? BN / 2 : 0) + wn * (Cfg::WN / 2) + (j % (TN / 2)) * 16;
    else b_rows[j] = wn * Cfg::WN + j * 16;
  }
  typename FragSel<BK, TM, BM, AKC>::type fa;
  typename FragSel<BK, TN, BN, BKC>::type fb;
  fa.init(lane, a_rows);
  fb.init(lane, b_rows);

  f32x4_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.f;

  auto issue = [&](int kt, uint32_t stage) {     // kt < 0: no stage left for this group, all zeros
    const int seg = SEGS ? (kt >= kt_per_seg ? 1 : 0) + (kt >= 2 * kt_per_seg ? 1 : 0) : 0;
    const int k0 = KG > 1 && kt < 0 ? 0 : (kt - seg * kt_per_seg) * BK;
    const int K = KG > 1 && kt < 0 ? 0 : p.K;
    const bool tail = k0 + BK > K;
    if (DUAL || !SEGS) {
      da.issue(ra0, ra0, stage, k0, K, tail);
      db.issue(rb0, rb1, stage + A_BYTES, k0, K, tail);
    } else {
      da.issue(select_rsrc(seg, ra0, ra1, ra2), ra0, stage, k0, K, tail);
      db.issue(select_rsrc(seg, rb0, rb1, rb2), rb0, stage + A_BYTES, k0, K, tail);
    }
  };

  // Fragments: A double-buffered by K step, B single-buffered -- a B block is reloaded for the next
  // step right behind the MFMAs of its column, the last use of its present contents.
  bf16x8_t af[2][TM], bfr[TN];
  // One 32-K step: MFMAs column by column; behind column j the loads of the next step's B block j and
  // (for j < TM) A block j from `next`, step `ns`.  (Behind the very last step of the K loop these
  // loads fetch fragments nobody uses: cheaper than a branch per column.)
  auto step = [&](int cur, const uint8_t* next, int ns) {
#pragma unroll
    for (int j = 0; j < TN; ++j) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[cur][i], bfr[j], acc[i][j], 0, 0, 0);
      bfr[j] = fb.fetch_one(j, next + A_BYTES, ns);
      if constexpr (TM <= TN) {
        if (j < TM) af[cur ^ 1][j] = fa.fetch_one(j, next, ns);
      } else {                 // taller than wide: the A blocks are shared out over the columns
#pragma unroll
        for (int i = j * TM / TN; i < (j + 1) * TM / TN; ++i) af[cur ^ 1][i] = fa.fetch_one(i, next, ns);
      }
    }
    // The scheduler's built-in pattern that alternates single MFMAs with single LDS reads.  Measured
    // against its other pattern, none, and an order pinned column by column (same card, alternating
    // runs): the large launches +4 to +9 %.
    __builtin_amdgcn_iglp_opt(1);
  };
  // The two waves that share a SIMD (w and w + 4) run the same instruction stream; a raised issue
  // priority for one of them keeps the pair slightly out of step, so that one tends to issue MFMAs
  // while the other waits on LDS.
  if (NT == 512 && wave >= 4) __builtin_amdgcn_s_setprio(1);
  const int nst = kt_end - kt_begin;
  // A group of one wave reads nothing but its own fills: it waits for itself only, and for no one within the K loop.
  constexpr bool SOLO = Cfg::NT == 64;
  auto meet = [&]() {
    if constexpr (SOLO) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // reads of the buffer that is refilled next
    else __syncthreads();
  };
  // stages of this group; of the one with the most where the groups meet in every turn
  const int turns = SOLO ? (nst - group + KG - 1) / KG : KG > 1 ? (nst + KG - 1) / KG : nst;
  // The (up to eight) tiles of a tile column run at the same time on one XCD and share their B panel.
  // Each starts its K loop at a different stage (rotation by the tile row, wrapping around), so that
  // they do not all ask L2 for the same lines at the same moment: the first request of a line then
  // misses and the others hit, instead of queueing behind the miss.  A rotation of one stage per tile
  // row keeps every shared line in use for at most eight stages, well inside the 4 MB L2 (larger
  // strides measured slower).  Measured on the 7B-shaped layer: recompute launch -3.5 %, the others
  // -1 % to 0.  The summation order over K depends on the tile row only, so reruns stay bit-equal.
  int rot = m0 / BM & 7;
  while (rot >= nst && rot > 0) rot = nst > 0 ? rot - nst : 0;
  auto kmap = [&](int turn) {
    const int i = KG > 1 ? turn * KG + group : turn;
    if (KG > 1 && i >= nst) return -1;
    int k = kt_begin + i + rot;
    return k >= kt_end ? k - nst : k;
  };
  // K-contiguous operands whose K is no multiple of 8: the last stage of a segment is cleaned in LDS once
  // it has landed, behind one more barrier (the bytes behind K may hold anything, also in one operand only).
  const bool ragged = RAGGED && (AKC || BKC) && (K & 7) && !p.kpad_ok;
  auto clear_ragged = [&](int kt, uint8_t* stage) {
    const int seg = (kt >= kt_per_seg ? 1 : 0) + (kt >= 2 * kt_per_seg ? 1 : 0);
    if (!ragged) return;
    const bool last = kt == (seg + 1) * kt_per_seg - 1;
    if ((KG == 1 || SOLO) && !last) return;      // several groups: every one of them meets the barrier in every turn
    if (last) {
      DmaA::clear_tail(stage, t, K % BK);
      DmaB::clear_tail(stage + A_BYTES, t, K % BK);
    }
    meet();
  };
  if (turns > 0) {
    // Fill every buffer of the ring, wait for the first stage only.
#pragma unroll
    for (int s = 0; s < NS; ++s)
      if (s < turns) issue(kmap(s), smem_addr + s * STAGE);
    wait_fills_leave<FPS>(min(NS, turns) - 1);
    meet();
    clear_ragged(kmap(0), smem);
#pragma unroll
    for (int i = 0; i < TM; ++i) af[0][i] = fa.fetch_one(i, smem, 0);
#pragma unroll
    for (int j = 0; j < TN; ++j) bfr[j] = fb.fetch_one(j, smem + A_BYTES, 0);
    int buf = 0;
    static_assert(KS == 2, "two 32-K steps per stage");
    for (int turn = 0; turn < turns; ++turn) {
      const uint8_t* sc = smem + buf * STAGE;
      const int nbuf = buf + 1 == NS ? 0 : buf + 1;
      step(0, sc, 1);
      // Every fragment of this stage is in registers or on its way.  Wait for the next stage only
      // (younger fills stay in flight), meet the other waves, then refill this buffer NS stages ahead.
      wait_fills_leave<FPS>(min(NS - 2, turns - turn - 2));
      meet();
      if (turn + NS < turns) issue(kmap(turn + NS), smem_addr + buf * STAGE);
      if (ragged && turn + 1 < turns) clear_ragged(kmap(turn + 1), smem + nbuf * STAGE);
      step(1, smem + nbuf * STAGE, 0);
      buf = nbuf;
    }
  }

  // The groups' tiles are added in a fixed order, lane by lane (the buffers are free: the last barrier followed
  // every fragment fetch that is used); the first group goes on to the epilogue.
  if constexpr (KG > 1) {
    f32x4_t* part = (f32x4_t*)(smem_all + Pipe::NW * Pipe::EP_WAVE_BYTES);
    __syncthreads();
    if (group > 0) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) part[(((group - 1) * TM + i) * TN + j) * NT + t] = acc[i][j];
    }
    __syncthreads();
    if (group > 0) return;
#pragma unroll
    for (int g = 1; g < KG; ++g)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] += part[(((g - 1) * TM + i) * TN + j) * NT + t];
  }

  fold_norm<EPI>(p, lane);
  // Epilogue, staged through LDS so that global accesses are 16 bytes per lane and cover whole
  // rows (bf16: eight columns per access, fp32: two accesses of four).  Accumulator element e of a 16x16 block sits at row
  // 4*(lane/16) + e, column lane%16; each wave writes 32 rows of its sub-tile as fp32
  // into its own LDS slice (row stride RS floats, chosen so that the 16-lane groups hit
  // different banks), then reads rows back eight columns per lane.  The operand stages are
  // free at this point: the loop's last barrier followed every fragment fetch and every fill.
  {
    constexpr int TNO = DUAL ? TN / 2 : TN;
    constexpr int W = TNO * 16;                 // columns per matrix in this wave's sub-tile
    constexpr int RS = W + 4;                   // 4*RS % 64 == 16: the four row groups of a store, and neighbouring rows of a read, fall on different banks
    constexpr int MAT = 32 * RS;                // floats per staged matrix
    float* ep = (float*)(smem + wave * Pipe::EP_WAVE_BYTES);
    const int wr_off = (4 * (lane >> 4)) * RS + (lane & 15);
    constexpr int LPR = W / 8;                  // lanes per row when reading back
    constexpr int RPI = 64 / LPR;               // rows per read instruction
    const int rd_row = lane / LPR, rd_c8 = (lane % LPR) * 8;
    const int row_w = m0 + wm * Cfg::WM;
    const int col_w = n0 + wn * (DUAL ? Cfg::WN / 2 : Cfg::WN) + rd_c8;
#pragma unroll
    for (int i = 0; i < TM / 2; ++i) {        // 32 rows = two block rows at a time
#pragma unroll
      for (int ih = 0; ih < 2; ++ih)
#pragma unroll
        for (int j = 0; j < TNO; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int o = wr_off + (16 * ih + e) * RS + j * 16;
            ep[o] = acc[2 * i + ih][j][e];
            if constexpr (DUAL) ep[MAT + o] = acc[2 * i + ih][j + TN / 2][e];
          }
      // fp32 outputs: four columns per lane, so that one store instruction covers whole 512-byte row
      // pieces (with eight columns per lane each of the two 16-byte stores would fill every other
      // 16 bytes of its lines)
      constexpr bool F32_OUT = EPI == EPI_HILO;
      if constexpr (F32_OUT || EPI == EPI_GRAD || EPI == EPI_STORE) {
        if (F32_OUT || (EPI == EPI_GRAD ? head.out_f32 != 0 : p.splits > 1)) {
          constexpr int LPR4 = W / 4, RPI4 = 64 / LPR4;
          const int r4 = lane / LPR4, c4 = (lane % LPR4) * 4;
#pragma unroll
          for (int it = 0; it < 32 / RPI4; ++it) {
            const int rl = it * RPI4 + r4;
            const f32x4_t g = *(const f32x4_t*)(ep + rl * RS + c4);
            const float v4[4] = {g[0], g[1], g[2], g[3]};
            epilogue_vec4<EPI>(p, head, split, row_w + i * 32 + rl, col_w - rd_c8 + c4, v4);
          }
          continue;
        }
      }
#pragma unroll
      for (int it = 0; it < (F32_OUT ? 0 : 32 / RPI); ++it) {
        const int rl = it * RPI + rd_row;
        const float* src = ep + rl * RS + rd_c8;
        float v[8], v2[8];
        const f32x4_t g0 = *(const f32x4_t*)src, g1 = *(const f32x4_t*)(src + 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) { v[e] = g0[e]; v[4 + e] = g1[e]; v2[e] = 0.f; v2[4 + e] = 0.f; }
        if constexpr (DUAL) {
          const f32x4_t z0 = *(const f32x4_t*)(src + MAT), z1 = *(const f32x4_t*)(src + MAT + 4);
#pragma unroll
          for (int e = 0; e < 4; ++e) { v2[e] = z0[e]; v2[4 + e] = z1[e]; }
        }
        if constexpr (EPI == EPI_ROPE) {     // the wave's columns are whole heads: the other half of the pairs is in its slice
          if (p.rope_half) {
            const float* other = ep + rl * RS + (rd_c8 ^ p.rope_half);
            const f32x4_t z0 = *(const f32x4_t*)other, z1 = *(const f32x4_t*)(other + 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) { v2[e] = z0[e]; v2[4 + e] = z1[e]; }
          }
        }
        if constexpr (!F32_OUT) epilogue_vec8<EPI>(p, head, split, row_w + i * 32 + rl, col_w, v, v2);
      }
    }
  }
}

// Measurement only: shader-clock cycles and constant-rate (100 MHz) ticks of a workgroup.
struct WorkgroupClock {
  uint64_t c0 = 0, w0 = 0;
  __device__ inline void start(const KHead& head) {
    if (head.clk) { c0 = clock64(); w0 = wall_clock64(); }
  }
  __device__ inline void stop(const KHead& head) const {
    if (head.clk && (blockIdx.x & 63) == 0 && threadIdx.x == 0) {
      uint32_t* o = head.clk + 2 * ((blockIdx.x >> 6) & 63);
      o[0] = (uint32_t)(clock64() - c0);
      o[1] = (uint32_t)(wall_clock64() - w0);
    }
  }
};

template <class Cfg, class Pipe, bool AKC, bool BKC, int EPI, bool RAGGED>
__global__ __launch_bounds__(Pipe::THREADS, 2) void gemm_bf16_dtl_kernel(const KArgs args) {
  constexpr int BM = Cfg::BM, BN_OUT = epi_is_dual(EPI) ? Cfg::BN / 2 : Cfg::BN;
  extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
  const KHead head = load_head();
  if constexpr (side_kind(AKC, BKC, EPI) != SIDE_NONE) {
    if ((int)blockIdx.x >= head.gemm_blocks) {
      run_side<__bf16, side_kind(AKC, BKC, EPI)>(args, blockIdx.x - head.gemm_blocks, smem);
      return;
    }
  }
  WorkgroupClock clock;
  clock.start(head);
  int index;
  const int prob = map_problem(head, blockIdx.x, &index);
  const KProblem kp = load_problem(prob);
  const TileCoord tc = map_tile<BM, BN_OUT>(head, kp, prob, index);
  const GemmProblem p = product_view<2>(head, kp, tc.z);
  const int m0 = tc.tm * BM, n0 = tc.tn * BN_OUT;
  if (causal_tile_unused(p, m0, n0, BM)) return;
  dtl_tile<Cfg, Pipe, AKC, BKC, EPI, RAGGED, true>(head, p, m0, n0, tc.split, smem);
  clock.stop(head);
}

// The recompute with the SwiGLU backward (problem 0, dual) and the dA = dY Wd (problem 1) that its epilogue reads, tile by
// tile in one workgroup: a launch less for calls of few tiles.  dA goes through memory as between the two launches, from
// and to the same lane; its tile has the recompute's rows and half its columns, in waves that hold the same elements.
// K = d is a multiple of 8 in both.
template <class C1, class P1, class C2, class P2>
__global__ __launch_bounds__(P2::THREADS, 2) void gemm_bf16_pair_kernel(const KArgs args) {
  static_assert(P1::THREADS == P2::THREADS && P1::LDS_BYTES <= P2::LDS_BYTES && C1::BM == C2::BM && 2 * C1::BN == C2::BN &&
                C1::WAVES_M == C2::WAVES_M && C1::WAVES_N == C2::WAVES_N, "the same outputs");
  extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
  const KHead head = load_head();
  const KProblem kp = load_problem(0), kd = load_problem(1);
  const TileCoord tc = map_tile<C1::BM, C1::BN>(head, kp, 0, xcd_remap(blockIdx.x, head.total));
  const int m0 = tc.tm * C1::BM, n0 = tc.tn * C1::BN;
  dtl_tile<C1, P1, true, false, EPI_STORE, false, false>(head, product_view<2>(head, kd, 0), m0, n0, 0, smem);
  __syncthreads();      // the second product fills the LDS that the first one's epilogue reads
  dtl_tile<C2, P2, true, true, EPI_SWIGLU_BWD, false, false>(head, product_view<2>(head, kp, 0), m0, n0, 0, smem);
}

// Launches whose 256 x 256 tiles leave a last round of at most 128: the workgroups of the full rounds compute such
// tiles (Cfg), and the last round's tiles are shared out over the chip in halves, quarters or sixteenths (C2, C4, C16),
// which walk K two to six times as fast.  head.total counts the workgroups of the full rounds, the tail's tiles are the
// last of the problem with the most.
template <class Cfg, class Pipe, class C2, class P2, class C4, class P4, class C16, class P16, bool AKC, bool BKC, int EPI>
__global__ __launch_bounds__(Pipe::THREADS, 2) void gemm_bf16_tail_kernel(const KArgs args) {
  static_assert(P2::THREADS == Pipe::THREADS && P4::THREADS == Pipe::THREADS && P16::THREADS == Pipe::THREADS, "one launch");
  constexpr int BM = Cfg::BM, BN_OUT = epi_is_dual(EPI) ? Cfg::BN / 2 : Cfg::BN;
  extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
  const KHead head = load_head();
  if constexpr (side_kind(AKC, BKC, EPI) != SIDE_NONE) {
    if ((int)blockIdx.x >= head.gemm_blocks) {
      run_side<__bf16, side_kind(AKC, BKC, EPI)>(args, blockIdx.x - head.gemm_blocks, smem);
      return;
    }
  }
  WorkgroupClock clock;
  clock.start(head);
  const int bid = blockIdx.x, extra = bid - head.total;
  if (extra < 0) {
    int index;
    const int prob = map_problem(head, bid, &index);
    const KProblem kp = load_problem(prob);
    const TileCoord tc = map_tile<BM, BN_OUT>(head, kp, prob, index);
    const GemmProblem p = product_view<2>(head, kp, 0);
    dtl_tile<Cfg, Pipe, AKC, BKC, EPI, false, false>(head, p, tc.tm * BM, tc.tn * BN_OUT, 0, smem);
    clock.stop(head);
    return;
  }
  const int prob = head.tail >> 28, shift = head.tail >> 24 & 15, first = head.tail & 0xFFFFFF;
  const int e = xcd_remap(extra, head.gemm_blocks - head.total);
  const KProblem kp = load_problem(prob);
  const TileCoord tc = map_tile<BM, BN_OUT>(head, kp, prob, first + (e >> shift));
  const GemmProblem p = product_view<2>(head, kp, 0);
  const int part = e & ((1 << shift) - 1);
  int m0 = tc.tm * BM, n0 = tc.tn * BN_OUT;
  if (shift == 1) {
    m0 += part * C2::BM;
    if (m0 < p.M) dtl_tile<C2, P2, AKC, BKC, EPI, false, false>(head, p, m0, n0, 0, smem);
  } else if (shift == 2) {
    m0 += (part >> 1) * C4::BM;
    n0 += (part & 1) * (BN_OUT / 2);
    if (m0 < p.M && n0 < p.N) dtl_tile<C4, P4, AKC, BKC, EPI, false, false>(head, p, m0, n0, 0, smem);
  } else {
    m0 += (part >> 2) * C16::BM;
    n0 += (part & 3) * (BN_OUT / 4);
    if (m0 < p.M && n0 < p.N) dtl_tile<C16, P16, AKC, BKC, EPI, false, false>(head, p, m0, n0, 0, smem);
  }
}

}  // namespace mecefo
