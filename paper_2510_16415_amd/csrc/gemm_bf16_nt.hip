// bf16 GEMM instantiations with both operands K-contiguous: FFN recompute (U Wg^T, U Wu^T
// with SwiGLU epilogues), the down projection, the expand step C P^T of Eq. (2), and the
// attention-score products Q K^T and dO V^T of the standard-mode backward.
#include "gemm_bf16_launch.hip.h"
namespace mecefo {
// The rotation pairs columns of one head: a wave of the epilogue must hold whole heads, which the 128 columns
// of a 256 x 256 tile's wave and the 64 of a 128 x 128 one do for head dimensions 64 and 128 or 64.
// The rotation as a launch of its own takes 4 to 6 us with the gap in front of it on small calls, 17 for [3584 x 3584]: a tile
// that can rotate is taken when the model puts it within 6 us of the best one (an 8-layer stack of
// d = 512, 2048 tokens, whose 64 x 64 and 128 x 128 tiles are a tie: 1201 -> 1183 us).  Forwards with no allowance and
// with no limit against this one, us, two launches for the rotation then: 64 tokens, two heads of 64: 38.9 / 33.4 against 33.5; 256 tokens, eight of 64:
// 48.6 / 50.9 against 50.9 (the one where it costs); 2048 tokens, eight of 64: 63.0 / 61.5 against 61.5; 256 tokens, four
// of 128: 48.3 / 60.3 against 48.3; 512 tokens, sixteen of 128: 141 / 173 against 141.
// The best one is looked for among the tiles that a rotating launch is costed with.  A plain launch may be shorter, with its
// last round cut up, on 192-row or 32-row tiles: forwards that rotate against that, us: [1024 x 2944], heads of 64: 141 / 133;
// [3072 x 2048], 64: 187 / 177; [2816 x 1920], 64: 163 / 163; [5632 x 3072], 64: 541 / 518; [7936 x 2304], 128: 475 / 470.
// But the rotation behind it rounds Q and K to bf16 a second time, which the one on the fp32 accumulators does not (their
// error times sqrt 2), so that is not weighed against a few percent of time.
int gemm_bf16_rope_tile(const GemmLaunch& g, int dh) {
  const int forced = bf16_forced_tile();
  if (forced >= 0)
    return (forced == TILE_L && (dh == 64 || dh == 128)) || (dh == 64 && (forced == TILE_M2 || forced == TILE_M4)) ? forced : -1;
  if (dh != 64 && dh != 128) return -1;
  GemmLaunch rot = g;      // costed as what would go out: a launch that rotates has no last round that is cut up
  rot.epi = EPI_ROPE;
  int best = TILE_L;
  for (int c : {TILE_M2, TILE_M4})
    if (dh == 64 && bf16_tile_cost(rot, c) < bf16_tile_cost(rot, best)) best = c;
  float least;
  bf16_best_tile(rot, &least);
  return bf16_tile_cost(rot, best) <= least + 6.f ? best : -1;
}
static hipError_t run_rope(GemmLaunch& g, hipStream_t s) {
  switch (g.tile) {
    case TILE_L: return run_bf16<CfgL8, true, true, EPI_ROPE, PipeL, false>(g, s);
    case TILE_M2: return run_bf16<CfgM, true, true, EPI_ROPE, PipeM2>(g, s);
    case TILE_M4: return run_bf16<CfgM8, true, true, EPI_ROPE, PipeM4>(g, s);
    default: return hipErrorInvalidValue;
  }
}
template <class C2, class P2> struct PairKernel {
  using C1 = TileCfg<C2::BM, C2::BN / 2, C2::WAVES_M, C2::WAVES_N>;
  using P1 = DtlPipe<C1, P2::NS, P2::KG>;
  static hipError_t prepare() {
    static LdsLimitOnce limit;
    return limit.ensure((const void*)gemm_bf16_pair_kernel<C1, P1, C2, P2>, P2::LDS_BYTES);
  }
  static hipError_t run(const GemmLaunch& dA, const GemmLaunch& rec, hipStream_t s) {
    KArgs a, b;
    fill_kargs(a, rec, C1::BM, C1::BN, kBK);
    fill_kargs(b, dA, C1::BM, C1::BN, kBK);
    a.p[1] = b.p[0];
    if (a.h.total == 0) return hipSuccess;
    const hipError_t e = prepare();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((gemm_bf16_pair_kernel<C1, P1, C2, P2>), dim3(a.h.total), dim3(P2::THREADS), P2::LDS_BYTES, s, a);
    return hipGetLastError();
  }
};
// FFN backwards with two launches and with one, us, [tokens x d], f: [16 x 256], 128: 23.6 / 20.1; [129 x 512], 200: 23.2 /
// 20.7; [256 x 1024], 1000: 37.1 / 35.0; [777 x 768], 700: 35.3 / 32.4; [2048 x 512], 1376: 61.8 / 55.6; [1024 x 1024], 2736: 87.7
// / 82.7; [4096 x 1024], 1024: 89.1 / 84.6: the one launch takes 2 to 5 us less than the model says, on 64 x 64 tiles 0
// to 2.  Not so where the two
// go out on 32 x 32 tiles, with twice as many workgroups to share out K ([128 x 1024], 1024: 28.6 / 28.9), or on ones of 192 and
// 256 rows, which take fewer bytes ([2048 x 1024], 2736: 120.5 / 126.4; [2048 x 768], 2050: 92.2 / 95.7).
int gemm_bf16_pair_tile(const GemmLaunch& dA, const GemmLaunch& rec, float cost) {
  if (bf16_forced_tile() >= 0) return -1;
  float t1, t2;
  const int c1 = bf16_best_tile(dA, &t1), c2 = bf16_best_tile(rec, &t2);
  auto same = [](int c) { return c == TILE_M2 || c == TILE_M4 || c == TILE_T || c == TILE_T2; };
  const bool alike = same(c1) && same(c2);
  // the first product's stages move half the columns of B: three quarters of the recompute's bytes
  GemmLaunch both = rec;
  both.p[0].K += dA.p[0].K / 4 * 3;
  float t = t1 + t2;
  int best = -1;
  for (int c : {TILE_M2, TILE_M4, TILE_T, TILE_T2}) {
    const float x = bf16_tile_cost(both, c) + cost + (!alike ? 1.4f : c == TILE_M2 || c == TILE_M4 ? -2.f : 0.5f);
    if (x < t) { t = x; best = c; }
  }
  return best;
}
hipError_t launch_gemm_bf16_pair(const GemmLaunch& dA, const GemmLaunch& rec, int tile, hipStream_t s) {
  switch (tile) {
    case TILE_M2: return PairKernel<CfgM, PipeM2>::run(dA, rec, s);
    case TILE_M4: return PairKernel<CfgM8, PipeM4>::run(dA, rec, s);
    case TILE_T: return PairKernel<CfgT, PipeT>::run(dA, rec, s);
    case TILE_T2: return PairKernel<CfgT, PipeT2>::run(dA, rec, s);
    default: return hipErrorInvalidValue;
  }
}
hipError_t launch_gemm_bf16_nt(GemmLaunch& g, hipStream_t s) {
  switch (g.epi) {
    case EPI_STORE: return run_bf16_auto<true, true, EPI_STORE>(g, s);
    case EPI_GRAD: return run_bf16_auto<true, true, EPI_GRAD>(g, s);
    case EPI_SWIGLU_FWD: return run_bf16_auto<true, true, EPI_SWIGLU_FWD>(g, s);
    case EPI_SWIGLU_BWD: return run_bf16_auto<true, true, EPI_SWIGLU_BWD>(g, s);
    case EPI_ATTN_P: return run_bf16_auto<true, true, EPI_ATTN_P>(g, s);
    case EPI_ATTN_DS: return run_bf16_auto<true, true, EPI_ATTN_DS>(g, s);
    case EPI_POLY: return run_bf16_auto<true, true, EPI_POLY>(g, s);
    case EPI_HILO: return run_bf16_auto<true, true, EPI_HILO>(g, s);
    case EPI_RESID: return run_bf16_auto<true, true, EPI_RESID>(g, s);
    case EPI_ROPE: return run_rope(g, s);
    default: return hipErrorInvalidValue;
  }
}
hipError_t prepare_gemm_bf16_nt() {
  hipError_t e = hipSuccess;
  if (e == hipSuccess) e = prepare_bf16<true, true, EPI_STORE>();
  if (e == hipSuccess) e = prepare_bf16<true, true, EPI_GRAD>();
  if (e == hipSuccess) e = prepare_bf16<true, true, EPI_SWIGLU_FWD>();
  if (e == hipSuccess) e = prepare_bf16<true, true, EPI_SWIGLU_BWD>();
  if (e == hipSuccess) e = prepare_bf16<true, true, EPI_ATTN_P>();
  if (e == hipSuccess) e = prepare_bf16<true, true, EPI_ATTN_DS>();
  if (e == hipSuccess) e = prepare_bf16<true, true, EPI_POLY>();
  if (e == hipSuccess) e = prepare_bf16<true, true, EPI_HILO>();
  if (e == hipSuccess) e = prepare_bf16<true, true, EPI_RESID>();
  if (e == hipSuccess) e = PairKernel<CfgM, PipeM2>::prepare();
  if (e == hipSuccess) e = PairKernel<CfgM8, PipeM4>::prepare();
  if (e == hipSuccess) e = PairKernel<CfgT, PipeT>::prepare();
  if (e == hipSuccess) e = PairKernel<CfgT, PipeT2>::prepare();
  if (e == hipSuccess) e = Bf16Kernel<CfgL8, true, true, EPI_ROPE, PipeL, false>::prepare();
  if (e == hipSuccess) e = Bf16Kernel<CfgM, true, true, EPI_ROPE, PipeM2, true>::prepare();
  if (e == hipSuccess) e = Bf16Kernel<CfgM8, true, true, EPI_ROPE, PipeM4, true>::prepare();
  return e;
}
}  // namespace mecefo
