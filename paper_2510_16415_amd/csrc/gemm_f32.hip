// fp32 GEMM for the fp32 storage path (small reference-precision config) on v_mfma_f32_16x16x4_f32: fp32
// operands, fp32 accumulation.  Layouts, K segments, dual products and epilogues mirror the bf16 core so that
// the host orchestration is identical for both dtypes.
//
// What bounds it: these products are small (256 tokens, d = 256, f = 688: 16 to 44 tiles of 64 x 64 for 256
// CUs), so the length of one workgroup's walk along K is the launch's time.  Hence 32 x 32 tiles with K stages of
// 64, whose global loads (four elements each) are issued a stage ahead into registers, two LDS buffers (one
// barrier per stage), and the four waves share out the K of a stage (16 each) instead of the tile; their partial
// tiles are added through LDS in a fixed order.  Launches with 64 x 64 tiles for every CU take those, each wave
// a 32 x 32 quarter, K stages of 32: half the operand bytes per multiply-add.
// Measured against the kernel before (64 x 64 tiles of plain FMAs, K slices of 16, loads in front of their use):
// one layer's skip backward at the sizes above 574 -> 69 us, the exact FFN backward of 1024 tokens, d = 512,
// f = 1536 937 -> 217 us and of 2048 tokens, d = 2048, f = 5461 8258 -> 4001 us; errors against fp64 are the same
// (64 x 64 tiles) or half (the split sums) of what they were.
#include "gemm_bf16_dtl.hip.h"

#include <type_traits>

namespace mecefo {

namespace {

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4f_t;

// FT x FT output tile, K stages of FK; KSPLIT: the four waves share out K, else the tile; FAR: rows addressed in 64 bits.
template <int FT_, int FK_, bool KSPLIT_, bool FAR_ = false> struct F32Cfg {
  static constexpr int FT = FT_, FK = FK_;
  static constexpr bool KSPLIT = KSPLIT_, FAR = FAR_;
  static constexpr int FS = FK + 4;           // LDS row stride (floats): the 16 rows of an operand read fall on different banks
  static constexpr int NV = FT * FK / 1024;   // four-element loads per thread, operand and stage
};
using CfgSmall = F32Cfg<32, 64, true>;
using CfgWide = F32Cfg<64, 32, false>;
using CfgFar = F32Cfg<32, 64, true, true>;

// One operand tile, [FT rows][FK] in LDS.  A load takes four consecutive elements of the source's rows (dword
// alignment is enough): K-contiguous four K of a row, K-strided four rows of one K.  The buffer range is the
// matrix itself, so what lies behind its last element reads as zero; rows and K outside the matrix are pointed
// behind the range.  The offsets from the first row of a tile (or K row of a stage) are 32 bits wide, which every
// tensor below 2 GiB allows.  A projection's row stride is not bounded: rows that lie further apart are read element
// by element through 64-bit addresses (FAR).
template <class Cfg, bool kc>
struct TileF32 {
  static constexpr int NV = Cfg::NV, FT = Cfg::FT, FK = Cfg::FK;
  f32x4_t v[NV];
  uint32_t voff[NV];            // byte offsets within the tile's rows (K-contiguous) or the stage's K rows
  int64_t total, first, ld4;    // bytes of the matrix, bytes in front of the tile's first row, bytes per row
  int row0, rows;               // FAR
  __device__ inline int row(int t, int i) const { const int c = t + 256 * i; return kc ? c / (FK / 4) : c % (FT / 4) * 4; }
  __device__ inline int kk(int t, int i) const { const int c = t + 256 * i; return kc ? c % (FK / 4) * 4 : c / (FT / 4); }
  __device__ inline void init(int t, int64_t ld, int first_row, int n_rows, int K) {
    row0 = first_row;
    rows = n_rows;
    ld4 = ld * 4;
    if constexpr (Cfg::FAR) return;
    total = K > 0 ? (kc ? (rows - 1) * ld4 + K * (int64_t)4 : (K - 1) * ld4 + rows * (int64_t)4) : 0;
    first = kc ? row0 * ld4 : 0;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int r = row0 + row(t, i), k = kk(t, i);
      voff[i] = r < rows ? (uint32_t)((kc ? (int64_t)(r - row0) * ld + k : (int64_t)k * ld + r) * 4) : 0x80000000u;
    }
  }
  __device__ inline void load(const void* base, int t, int k0, int K) {
    if constexpr (Cfg::FAR) {
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        const int r = row0 + row(t, i), k = k0 + kk(t, i);
        const float* q = (const float*)((const char*)base + (kc ? (int64_t)r * ld4 + k * (int64_t)4 : (int64_t)k * ld4 + r * (int64_t)4));
#pragma unroll
        for (int e = 0; e < 4; ++e) v[i][e] = (kc ? r < rows && k + e < K : k < K && r + e < rows) ? q[e] : 0.f;
      }
      return;
    }
    const bool tail = k0 + FK > K;              // wave-uniform
    // the base moves with the tile (or stage): the matrix may be longer than the 2 GiB a buffer spans
    const int64_t at = kc ? first : k0 * ld4, left = total - at;
    const uint32_t soff = kc ? (uint32_t)k0 * 4 : 0;
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((char*)const_cast<void*>(base) + at, 0,
                                                                       (int)(left < 0x7FFFFFFF ? left : 0x7FFFFFFF), 0x00020000);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const uint32_t off = tail && k0 + kk(t, i) >= K ? 0x80000000u : voff[i];
      v[i] = __builtin_bit_cast(f32x4_t, (u32x4f_t)__builtin_amdgcn_raw_buffer_load_b128(r, off, soff, 0));
    }
  }
  // `left`: K of this stage and beyond.  Elements behind a ragged K are cleared here, not behind the load, which
  // would wait for it; elements behind a K-strided row end only reach outputs outside the matrix.
  __device__ inline void store(float* lds, int t, int left) {
    if (kc && left < FK) {
#pragma unroll
      for (int i = 0; i < NV; ++i)
#pragma unroll
        for (int e = 1; e < 4; ++e) v[i][e] = kk(t, i) + e < left ? v[i][e] : 0.f;
    }
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      float* d = lds + row(t, i) * Cfg::FS + kk(t, i);
      if constexpr (kc) {
        *(f32x4_t*)d = v[i];
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) d[e * Cfg::FS] = v[i][e];
      }
    }
  }
};

// Adds the four waves' partial 32 x 32 tiles through LDS in a fixed order ([wave][matrix][32][33]) and stores them.
// Accumulator element e of a 16x16 block is row 4 (lane / 16) + e, column lane % 16.
template <int EPI, int NB>
__device__ inline void sum_quarters(const GemmProblem& p, const KHead& head, int split, int m0, int n0, int t,
                                    const f32x4_t (&acc)[NB][2][2], float* part) {
  constexpr int FT = 32;
  const int lane = t & 63, wave = t >> 6;
#pragma unroll
  for (int w = 0; w < NB; ++w)
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          part[((wave * NB + w) * FT + 16 * i + 4 * (lane >> 4) + e) * (FT + 1) + 16 * j + (lane & 15)] = acc[w][i][j][e];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < FT * FT / 256; ++i) {
    const int r = (t + 256 * i) / FT, c = t % FT;
    float s[2] = {0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NB; ++w) {
      const float* q = part + (w * FT + r) * (FT + 1) + c;
      constexpr int W = NB * FT * (FT + 1);      // one wave's partial tiles
      s[w] = (q[0] + q[W]) + (q[2 * W] + q[3 * W]);
    }
    epilogue_elem<EPI, float>(p, head, split, m0 + r, n0 + c, s[0], s[1]);
  }
}

template <class Cfg, int EPI, bool AKC, bool BKC>
__global__ __launch_bounds__(256, 2) void gemm_f32_kernel(const KArgs args) {
  constexpr bool DUAL = epi_is_dual(EPI);
  constexpr int FT = Cfg::FT, FK = Cfg::FK, FS = Cfg::FS;
  constexpr int NB = DUAL ? 2 : 1, MATS = 1 + NB;
  constexpr int KG = Cfg::KSPLIT ? FK / 64 : FK / 16;       // groups of 16 K per wave and stage
  __shared__ __attribute__((aligned(16))) float lds[2][MATS][FT * FS];
  static_assert(!Cfg::KSPLIT || 4 * NB * FT * (FT + 1) <= 2 * MATS * FT * FS, "the partial tiles reuse the operand buffers");
  const KHead head = load_head();
  if constexpr (side_kind(AKC, BKC, EPI) != SIDE_NONE) {
    if ((int)blockIdx.x >= head.gemm_blocks) {
      run_side<float, side_kind(AKC, BKC, EPI)>(args, blockIdx.x - head.gemm_blocks, &lds[0][0][0]);
      return;
    }
  }
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  int index;
  const int prob = map_problem(head, blockIdx.x, &index);
  const KProblem kp = load_problem(prob);
  const TileCoord tc = map_tile<FT, FT>(head, kp, prob, index);
  const GemmProblem p = product_view<4>(head, kp, tc.z);
  const int m0 = tc.tm * FT, n0 = tc.tn * FT;
  if (causal_tile_unused(p, m0, n0, FT)) return;
  const int nseg = DUAL ? 1 : p.nseg;
  const int kt_per_seg = (uint32_t)(p.K + FK - 1) / FK;
  const int kt_total = kt_per_seg * nseg;
  int kt_begin = tc.split * p.chunk;
  int kt_end = min(kt_total, kt_begin + p.chunk);
  causal_clip(p, m0, n0, FT, FK, kt_begin, kt_end);

  f32x4_t acc[NB][2][2];
#pragma unroll
  for (int w = 0; w < NB; ++w)
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[w][i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  TileF32<Cfg, AKC> ta;
  TileF32<Cfg, BKC> tb[NB];
  ta.init(t, p.lda, m0, p.M, p.K);
#pragma unroll
  for (int w = 0; w < NB; ++w) tb[w].init(t, p.ldb, n0, p.N, p.K);
  auto load = [&](int kt) {
    const int seg = (kt >= kt_per_seg ? 1 : 0) + (kt >= 2 * kt_per_seg ? 1 : 0);
    const int k0 = (kt - seg * kt_per_seg) * FK;
    ta.load(DUAL ? p.A[0] : select_base(seg, p.A[0], p.A[1], p.A[2]), t, k0, p.K);
    tb[0].load(DUAL ? p.B[0] : select_base(seg, p.B[0], p.B[1], p.B[2]), t, k0, p.K);
    if constexpr (DUAL) tb[NB - 1].load(p.B[1], t, k0, p.K);
  };
  if (kt_begin < kt_end) load(kt_begin);
  // operand reads: lane holds row lane % 16 and four consecutive K, 4 (lane / 16) .. + 3 of a group of 16; MFMA
  // step e takes element e of both operands (K in another order, the same for both)
  const int wm = Cfg::KSPLIT ? 0 : wave >> 1, wn = Cfg::KSPLIT ? 0 : wave & 1;
  const int lane_off = (lane & 15) * FS + 4 * (lane >> 4) + (Cfg::KSPLIT ? 16 * wave : 0);
  const int a_off = lane_off + wm * 32 * FS, b_off = lane_off + wn * 32 * FS;
  for (int kt = kt_begin; kt < kt_end; ++kt) {
    float(*buf)[FT * FS] = lds[(kt - kt_begin) & 1];
    const int seg = (kt >= kt_per_seg ? 1 : 0) + (kt >= 2 * kt_per_seg ? 1 : 0);
    const int left = p.K - (kt - seg * kt_per_seg) * FK;
    ta.store(buf[0], t, left);
#pragma unroll
    for (int w = 0; w < NB; ++w) tb[w].store(buf[1 + w], t, left);
    if (kt + 1 < kt_end) load(kt + 1);
    // one barrier per stage: whoever read this buffer two stages ago has passed the previous one
    __syncthreads();
#pragma unroll
    for (int g = 0; g < KG; ++g) {
      f32x4_t a[2], b[NB][2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        a[i] = *(const f32x4_t*)(buf[0] + a_off + 16 * i * FS + 16 * g);
#pragma unroll
        for (int w = 0; w < NB; ++w) b[w][i] = *(const f32x4_t*)(buf[1 + w] + b_off + 16 * i * FS + 16 * g);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int w = 0; w < NB; ++w)
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
              acc[w][i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][e], b[w][j][e], acc[w][i][j], 0, 0, 0);
    }
  }
  // accumulator element e of a 16x16 block is row 4 (lane / 16) + e, column lane % 16
  if constexpr (!Cfg::KSPLIT) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          epilogue_elem<EPI, float>(p, head, tc.split, m0 + 32 * wm + 16 * i + 4 * (lane >> 4) + e,
                                    n0 + 32 * wn + 16 * j + (lane & 15), acc[0][i][j][e], acc[NB - 1][i][j][e]);
    return;
  }
  __syncthreads();
  sum_quarters<EPI>(p, head, tc.split, m0, n0, t, acc, &lds[0][0][0]);
}

// The 32 x 32 tile with operands that go straight to LDS.  One stage ahead in registers, as above, a K stage takes the
// latency of its loads, 0.75 us; a ring of six stages of 16 KiB (five of 24 for dual products) filled by
// `buffer_load_dwordx4 ... lds` has 80 KiB and more in flight, and the matrix cores set the pace (16 MFMAs of 32 clocks
// per wave and stage, 0.21 us).  Same tiles, same K order, so the sums are those of the kernel above bit for bit.
// Needs rows that start on 16 bytes and whole pieces along a contiguous K (f32_direct); a piece that reaches behind the
// end of K-strided rows brings elements that only outputs outside the matrix see.  256 tokens, d = 256, f = 688, skip
// backward: 57.1 -> 51.9 us.
// K-contiguous operands: [32 rows][64 K], the 16-byte chunks of a row XOR-swizzled by it.  K-strided ones: [64 K][32 rows]
// in memory order; a lane reads single elements, 16 rows of four K rows at once, and neither the K row's parity nor its
// half of the 32 rows may be the same for two of them: K bit 2 is folded into bit 0, K bit 3 into the chunk.
template <bool kc>
struct DmaF32 {
  uint32_t voff[2];
  int at;            // K-contiguous: first K of the chunk; K-strided: K row of instruction 0
  int w;
  __device__ inline void init(int lane, int wave, int64_t ld, int row0, int rows) {
    w = wave;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int i = 4 * q + w;
      if constexpr (kc) {
        const int r = 4 * i + (lane >> 4);
        at = 4 * ((lane & 15) ^ (r & 15));                    // the same for both: 16 rows apart
        voff[q] = row0 + r < rows ? ((uint32_t)(row0 + r) * (uint32_t)ld + at) * 4 : kOOB;
      } else {
        const int pk = 8 * w + (lane >> 3), c = (lane & 7) ^ (4 * (w & 1));
        at = pk ^ (pk >> 2 & 1);
        voff[q] = row0 + 4 * c < rows ? ((uint32_t)(at + 32 * q) * (uint32_t)ld + row0 + 4 * c) * 4 : kOOB;
      }
    }
  }
  // soff: bytes to the stage; left: K from its start on (wave-uniform)
  __device__ inline void issue(u32x4_t r, uint32_t tile, uint32_t soff, int left) const {
    if (left >= 64) {
#pragma unroll
      for (int q = 0; q < 2; ++q) fill_lds_16B(r, tile + (4 * q + w) * 1024, voff[q], soff);
    } else {
#pragma unroll
      for (int q = 0; q < 2; ++q)
        fill_lds_16B(r, tile + (4 * q + w) * 1024, at + (kc ? 0 : 32 * q) < left ? voff[q] : kOOB, soff);
    }
  }
  // Block i of 16 rows for this wave's 16 K of a stage: element e of lane l is row l % 16, K 4 (l / 16) + e.
  static __device__ inline f32x4_t fetch(const uint8_t* tile, int lane, int wave, int i) {
    const int row = 16 * i + (lane & 15), g = lane >> 4;
    if constexpr (kc) return *(const f32x4_t*)(tile + row * 256 + (((4 * wave + g) ^ (row & 15)) << 4));
    f32x4_t v;
    const int col = (((row >> 2) ^ (4 * (g >> 1))) << 4) + (row & 3) * 4;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = *(const float*)(tile + (16 * wave + 4 * g + (e ^ (g & 1))) * 128 + col);
    return v;
  }
};

// Bytes of a matrix from its first to its last element.
inline int64_t f32_span(bool kc, int64_t ld, int rows, int K) {
  return K < 1 || rows < 1 ? 0 : kc ? ((rows - 1) * ld + K) * 4 : ((K - 1) * ld + rows) * 4;
}

template <int EPI> struct DirectF32 {
  static constexpr int NB = epi_is_dual(EPI) ? 2 : 1, NS = NB == 2 ? 5 : 6, TILE = 8192, STAGE = TILE * (1 + NB);
  static constexpr int LDS_BYTES = NS * STAGE;
  static_assert(4 * NB * 32 * 33 * 4 <= LDS_BYTES, "the partial tiles reuse the operand buffers");
};

template <int EPI, bool AKC, bool BKC>
__global__ __launch_bounds__(256, 2) void gemm_f32_direct_kernel(const KArgs args) {
  using D = DirectF32<EPI>;
  constexpr bool DUAL = epi_is_dual(EPI);
  constexpr int NB = D::NB, NS = D::NS, FT = 32, FK = 64, FPS = 2 * (1 + NB);
  extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
  const KHead head = load_head();
  if constexpr (side_kind(AKC, BKC, EPI) != SIDE_NONE) {
    if ((int)blockIdx.x >= head.gemm_blocks) {
      run_side<float, side_kind(AKC, BKC, EPI)>(args, blockIdx.x - head.gemm_blocks, smem);
      return;
    }
  }
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  int index;
  const int prob = map_problem(head, blockIdx.x, &index);
  const KProblem kp = load_problem(prob);
  const TileCoord tc = map_tile<FT, FT>(head, kp, prob, index);
  const GemmProblem p = product_view<4>(head, kp, tc.z);
  const int m0 = tc.tm * FT, n0 = tc.tn * FT;
  if (causal_tile_unused(p, m0, n0, FT)) return;
  const int nseg = DUAL ? 1 : p.nseg;
  const int kt_per_seg = (uint32_t)(p.K + FK - 1) / FK;
  int kt_begin = tc.split * p.chunk;
  int kt_end = min(kt_per_seg * nseg, kt_begin + p.chunk);
  causal_clip(p, m0, n0, FT, FK, kt_begin, kt_end);

  DmaF32<AKC> da;
  DmaF32<BKC> db;
  da.init(lane, wave, p.lda, m0, p.M);
  db.init(lane, wave, p.ldb, n0, p.N);
  // The next stage to be filled: a wave issues one instruction at a time, MFMAs included, and with one wave per SIMD
  // whatever it computes per stage adds to the stage, so the position is carried along.
  const uint32_t smem_addr = lds_address(smem);
  const uint32_t a_step = AKC ? 256u : 64u * (uint32_t)p.lda * 4, b_step = BKC ? 256u : 64u * (uint32_t)p.ldb * 4;
  int seg = (kt_begin >= kt_per_seg ? 1 : 0) + (kt_begin >= 2 * kt_per_seg ? 1 : 0);
  uint32_t at = (uint32_t)(kt_begin - seg * kt_per_seg);      // stage within the segment
  u32x4_t ra = make_rsrc_words(select_base(DUAL ? 0 : seg, p.A[0], p.A[1], p.A[2]));
  u32x4_t rb = make_rsrc_words(select_base(DUAL ? 0 : seg, p.B[0], p.B[1], p.B[2]));
  const u32x4_t rb1 = make_rsrc_words(p.B[1]);
  auto issue = [&](int slot) {
    const uint32_t stage = smem_addr + slot * D::STAGE;
    const int left = p.K - (int)at * FK;
    da.issue(ra, stage, at * a_step, left);
    db.issue(rb, stage + D::TILE, at * b_step, left);
    if constexpr (DUAL) db.issue(rb1, stage + 2 * D::TILE, at * b_step, left);
    if ((int)++at == kt_per_seg && !DUAL) {
      at = 0;
      ++seg;
      ra = make_rsrc_words(select_base(seg, p.A[0], p.A[1], p.A[2]));
      rb = make_rsrc_words(select_base(seg, p.B[0], p.B[1], p.B[2]));
    }
  };

  f32x4_t acc[NB][2][2];
#pragma unroll
  for (int w = 0; w < NB; ++w)
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[w][i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const int nst = kt_end - kt_begin;
#pragma unroll
  for (int s = 0; s < NS; ++s)
    if (s < nst) issue(s);
  // Operands of two stages: while the MFMAs run on one, the reads of the next are under way.
  struct Frags { f32x4_t a[2], b[NB][2]; } cur, next;
  auto fetch = [&](Frags& f, int slot) {
    const uint8_t* stage = smem + slot * D::STAGE;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      f.a[i] = DmaF32<AKC>::fetch(stage, lane, wave, i);
#pragma unroll
      for (int w = 0; w < NB; ++w) f.b[w][i] = DmaF32<BKC>::fetch(stage + (1 + w) * D::TILE, lane, wave, i);
    }
  };
  auto multiply = [&](const Frags& f) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int w = 0; w < NB; ++w)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            acc[w][i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(f.a[i][e], f.b[w][j][e], acc[w][i][j], 0, 0, 0);
  };
  // Behind this, stage k is in every wave's registers, its buffer is refilled NS stages ahead, and stage k + 1 has
  // landed; the younger ones stay in flight.
  int slot = 0;
  auto turn = [&](int k) {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (nst - k >= NS) asm volatile("s_waitcnt vmcnt(%0)" :: "n"((NS - 2) * FPS) : "memory");
    else wait_fills_leave<FPS>(nst - k - 2);
    __syncthreads();
    if (k + NS < nst) issue(slot);
    slot = slot + 1 == NS ? 0 : slot + 1;
  };
  if (nst > 0) {
    wait_fills_leave<FPS>(min(NS, nst) - 1);
    __syncthreads();
    fetch(cur, 0);
    for (int k = 0; k < nst; k += 2) {
      turn(k);
      if (k + 1 < nst) fetch(next, slot);
      multiply(cur);
      if (k + 1 == nst) break;
      turn(k + 1);
      if (k + 2 < nst) fetch(cur, slot);
      multiply(next);
    }
  }
  sum_quarters<EPI>(p, head, tc.split, m0, n0, t, acc, (float*)smem);
}

constexpr bool f32_nt_only(int epi) { return epi_is_dual(epi) || epi == EPI_ATTN_P || epi == EPI_ATTN_DS; }

// Workgroups of a launch with ft x ft tiles.
inline int f32_tiles(const GemmLaunch& g, int ft) {
  int tiles = 0;
  for (int i = 0; i < g.nprob; ++i)
    tiles += ((g.p[i].M + ft - 1) / ft) * ((g.p[i].N + ft - 1) / ft) * (g.p[i].batch > 1 ? g.p[i].batch : 1) *
             (g.p[i].splits > 1 ? g.p[i].splits : 1);
  return tiles;
}

template <class Cfg, int EPI>
hipError_t run_f32_cfg(GemmLaunch& g, hipStream_t stream) {
  KArgs a;
  fill_kargs(a, g, Cfg::FT, Cfg::FT, Cfg::FK);
  a.h.out_f32 = 1;
  a.h.clk = nullptr;
  if (a.h.total == 0) return hipSuccess;
  const dim3 grid(a.h.total + add_side(a, g, side_kind(g.a_kcontig, g.b_kcontig, EPI), 256));
  if (g.a_kcontig && g.b_kcontig) hipLaunchKernelGGL((gemm_f32_kernel<Cfg, EPI, true, true>), grid, dim3(256), 0, stream, a);
  else if constexpr (f32_nt_only(EPI)) return hipErrorInvalidValue;
  else if (g.a_kcontig) hipLaunchKernelGGL((gemm_f32_kernel<Cfg, EPI, true, false>), grid, dim3(256), 0, stream, a);
  else if (!g.b_kcontig) hipLaunchKernelGGL((gemm_f32_kernel<Cfg, EPI, false, false>), grid, dim3(256), 0, stream, a);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

// Whether every operand of the launch can go to LDS in 16-byte pieces: rows (and the products of a batch) that start on
// 16 bytes, whole pieces along a contiguous K, and less than 2 GiB.
inline bool f32_direct(const GemmLaunch& g) {
  const GemmProblem& f = g.p[0];
  if (f.batch > 1 && (f.a_bo | f.a_bi | f.b_bo | f.b_bi) % 4) return false;
  for (int i = 0; i < g.nprob; ++i) {
    const GemmProblem& p = g.p[i];
    const int segs = epi_is_dual(g.epi) ? 2 : p.nseg > 1 ? p.nseg : 1;
    uintptr_t bits = 0;
    for (int s = 0; s < segs; ++s) bits |= (uintptr_t)p.B[s] | (uintptr_t)p.A[epi_is_dual(g.epi) ? 0 : s];
    if (bits % 16 || p.lda % 4 || p.ldb % 4 || ((g.a_kcontig || g.b_kcontig) && p.K % 4)) return false;
    if (f32_span(g.a_kcontig, p.lda, p.M, p.K) >= (int64_t)1 << 31 || f32_span(g.b_kcontig, p.ldb, p.N, p.K) >= (int64_t)1 << 31) return false;
  }
  return true;
}

template <int EPI, bool AKC, bool BKC>
struct DirectKernelF32 {
  static hipError_t prepare() {
    static LdsLimitOnce limit;
    return limit.ensure((const void*)gemm_f32_direct_kernel<EPI, AKC, BKC>, DirectF32<EPI>::LDS_BYTES);
  }
  static hipError_t run(GemmLaunch& g, hipStream_t stream) {
    KArgs a;
    fill_kargs(a, g, 32, 32, 64);
    a.h.out_f32 = 1;
    a.h.clk = nullptr;
    if (a.h.total == 0) return hipSuccess;
    const hipError_t e = prepare();
    if (e != hipSuccess) return e;
    // a ring no longer than K needs, so that a CU takes more workgroups of a short one
    using D = DirectF32<EPI>;
    int stages = 1;
    for (int i = 0; i < g.nprob; ++i) stages = (a.p[i].chunk_nseg >> 2) > stages ? a.p[i].chunk_nseg >> 2 : stages;
    const unsigned side = add_side(a, g, side_kind(AKC, BKC, EPI), 256);
    const int ring = (stages < D::NS ? stages : D::NS) * D::STAGE, sum = 4 * D::NB * 32 * 33 * 4;
    hipLaunchKernelGGL((gemm_f32_direct_kernel<EPI, AKC, BKC>), dim3(a.h.total + side), dim3(256), ring > sum ? ring : sum, stream, a);
    return hipGetLastError();
  }
};
template <int EPI>
hipError_t run_f32_direct(GemmLaunch& g, hipStream_t stream) {
  if (g.a_kcontig && g.b_kcontig) return DirectKernelF32<EPI, true, true>::run(g, stream);
  if constexpr (!f32_nt_only(EPI)) {
    if (g.a_kcontig) return DirectKernelF32<EPI, true, false>::run(g, stream);
    if (!g.b_kcontig) return DirectKernelF32<EPI, false, false>::run(g, stream);
  }
  return hipErrorInvalidValue;
}
template <int... EPIS>
hipError_t prepare_f32() {
  hipError_t e = hipSuccess;
  auto one = [&](auto epi) {
    constexpr int E = decltype(epi)::value;
    if (e == hipSuccess) e = DirectKernelF32<E, true, true>::prepare();
    if constexpr (!f32_nt_only(E)) {
      if (e == hipSuccess) e = DirectKernelF32<E, true, false>::prepare();
      if (e == hipSuccess) e = DirectKernelF32<E, false, false>::prepare();
    }
  };
  (one(std::integral_constant<int, EPIS>{}), ...);
  return e;
}

// 64 x 64 tiles once they give every CU two workgroups.  Skip backwards of rank d / 4 to d / 8 with the line at 256 / 1024 / 2048
// tiles against 512, us: [1024 x 512], f 1376: 178 / 166 / 166 against 164; [4096 x 512], f 1376: 476 / 480 / 487 against
// 477; [4096 x 1024], f 2752: 1457 / 1458 / 1498 against 1457; [8192 x 256], f 688: 271 / 249 / 256 against 256.  Up to 1024 the
// smaller tiles are ahead where the launches that lie between are most of the call ([1024 x 1024], f 2752: 523 / 440 / 440
// against 474; [2048 x 512], f 1376: 297 / 262 / 262 against 278), behind where one of them is dU ([4096 x 512] with
// SIDE_OUTPUT: 476 / 495 / 505 against 476).
// Below that, 32 x 32 tiles, straight to LDS while the launch gives a CU at most two workgroups: its ring leaves room for one
// of them (two of short ones), and more of them run one after the other where the kernel with stages in registers has
// four at a time.  Direct to LDS against it, us: dU of [1024 x 1024], f 2752 (1024 tiles) 175 / 162, its token contraction
// of rank 256 (1632) 71 / 59, the recompute of [1024 x 512], f 1376 (1376) 52 / 42; but its projections (384) 13.8 / 19.4 and
// its dU (512) 46 / 49.  Skip backwards with the line at 512 tiles / 1024 / none: [512 x 512], f 1376: 99 / 107 / 107;
// [1024 x 512], f 1376: 162 / 167 / 189; [1024 x 1024], f 2752: 471 / 478 / 498; [2048 x 512], f 1376: 277 / 277 / 300.
template <int EPI>
hipError_t run_f32(GemmLaunch& g, hipStream_t stream) {
  if (f32_far(g)) {
    if constexpr (EPI == EPI_STORE || EPI == EPI_GRAD) return run_f32_cfg<CfgFar, EPI>(g, stream);
    else return hipErrorInvalidValue;
  }
  if (f32_tiles(g, 64) >= 512) return run_f32_cfg<CfgWide, EPI>(g, stream);
  return f32_tiles(g, 32) <= 2 * kCUs && f32_direct(g) ? run_f32_direct<EPI>(g, stream) : run_f32_cfg<CfgSmall, EPI>(g, stream);
}
}  // namespace

// dU of a small layer is a few dozen tiles that walk 2 f: with its parts added up by their reader the launch is as long as
// one of them.  A stage takes about 0.45 us, what a part costs its writer and reader 0.5 us.  256 tokens, d = 256, f = 688:
// three parts, the launch 14.3 -> 9.1 us.
void f32_plan_parts(GemmLaunch& g, int64_t room) {
  int at = -1, others = 0;
  for (int i = 0; i < g.nprob; ++i) {
    if (g.p[i].read_parts) at = i;
    else others += ((g.p[i].M + 31) / 32) * ((g.p[i].N + 31) / 32);
  }
  if (at < 0 || f32_tiles(g, 64) >= 512) return;
  GemmProblem& p = g.p[at];
  const int tiles = ((p.M + 31) / 32) * ((p.N + 31) / 32);
  const int stages = (p.K + 63) / 64 * (p.nseg > 1 ? p.nseg : 1);
  float best = 0.f;
  for (int s = 1; s <= kMaxNormParts && s <= stages; ++s) {
    if (s > 1 && ((int64_t)s * p.M * p.ldc > room || tiles * s + others > kCUs)) break;
    const float x = (float)((stages + s - 1) / s) * 0.45f + 0.5f * s;
    if (s == 1 || x < best) { best = x; p.splits = s; }
  }
}

// Whether the rows of one tile (K-contiguous operand) or the K rows of one stage span 2 GiB or more.  Only a
// projection can: it is B of the project products and A or B of the expand products.
bool f32_far(const GemmLaunch& g) {
  auto span = [](int64_t ld, int rows) { return ld * 4 * (rows < 64 ? rows : 64); };
  for (int i = 0; i < g.nprob; ++i) {
    const GemmProblem& p = g.p[i];
    if (span(p.lda, g.a_kcontig ? p.M : p.K) >= (int64_t)1 << 31 || span(p.ldb, g.b_kcontig ? p.N : p.K) >= (int64_t)1 << 31) return true;
  }
  return false;
}

// K splits of a launch that may be cut into up to `most` parts: a stage takes about 0.5 us while every CU has at
// most two workgroups, the sum of the parts one more launch of 5 us per problem.  Skip backwards never cut / always cut
// as far as the workspace holds, against this rule, us: [8192 x 128], f 344, rank 16: 189 / 133 against 133; [4096 x 256],
// f 688, rank 32: 198 / 182 against 182; [2048 x 128], f 344, rank 32: 79.0 / 78.0 against 79.0; [256 x 256], f 688: 69.5 / 74.8
// against 69.5; [1024 x 512], f 1376: 175 / 189 against 175; [4096 x 1024], f 2752: 1492 / 1501 against 1487.
void f32_plan_splits(GemmLaunch& g, int most) {
  const int tiles = f32_tiles(g, CfgSmall::FT);
  int stages = 0;
  for (int i = 0; i < g.nprob; ++i) {
    const int st = (g.p[i].K + CfgSmall::FK - 1) / CfgSmall::FK * (g.p[i].nseg > 1 ? g.p[i].nseg : 1);
    if (st > stages) stages = st;
  }
  int best = 1;
  float t = 0.f;
  for (int s = 1; s <= most && s <= (stages > 1 ? stages : 1); ++s) {
    const float n = (float)tiles * s / 512.f;
    const float x = (float)((stages + s - 1) / s) * 0.5f * (n > 1.f ? n : 1.f) + (s > 1 ? 5.f * g.nprob : 0.f);
    if (s == 1 || x < t) { t = x; best = s; }
  }
  for (int i = 0; i < g.nprob; ++i) g.p[i].splits = best;
}

hipError_t prepare_gemm_f32() {
  return prepare_f32<EPI_STORE, EPI_GRAD, EPI_SWIGLU_FWD, EPI_SWIGLU_BWD, EPI_ATTN_P, EPI_ATTN_DS, EPI_POLY, EPI_HILO, EPI_RESID>();
}

hipError_t launch_gemm_f32(GemmLaunch& g, hipStream_t s) {
  switch (g.epi) {
    case EPI_STORE: return run_f32<EPI_STORE>(g, s);
    case EPI_GRAD: return run_f32<EPI_GRAD>(g, s);
    case EPI_SWIGLU_FWD: return run_f32<EPI_SWIGLU_FWD>(g, s);
    case EPI_SWIGLU_BWD: return run_f32<EPI_SWIGLU_BWD>(g, s);
    case EPI_ATTN_P: return run_f32<EPI_ATTN_P>(g, s);
    case EPI_ATTN_DS: return run_f32<EPI_ATTN_DS>(g, s);
    case EPI_POLY: return run_f32<EPI_POLY>(g, s);
    case EPI_HILO: return run_f32<EPI_HILO>(g, s);
    case EPI_RESID: return run_f32<EPI_RESID>(g, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace mecefo
