// bf16 GEMM instantiations with both operands K-contiguous: FFN recompute (U Wg^T, U Wu^T
// with SwiGLU epilogues), the down projection, the expand step C P^T of Eq. (2), and the
// attention-score products Q K^T and dO V^T of the standard-mode backward.
#include "gemm_bf16_launch.hip.h"
namespace mecefo {
// The rotation pairs columns of one head: a wave of the epilogue must hold whole heads, which the 128 columns
// of a 256 x 256 tile's wave and the 64 of a 128 x 128 one do for head dimensions 64 and 128 or 64.
// The two rotations as launches cost about 7 us in all on small calls (3.4 us each and the gap), more on large
// ones: a tile that can rotate is taken when the model puts it within 6 us of the best one (an 8-layer stack of
// d = 512, 2048 tokens, whose 64 x 64 and 128 x 128 tiles are a tie: 1201 -> 1183 us).  Forwards with no allowance and
// with no limit against this one, us: 64 tokens, two heads of 64: 38.9 / 33.4 against 33.5; 256 tokens, eight of 64:
// 48.6 / 50.9 against 50.9 (the one where it costs); 2048 tokens, eight of 64: 63.0 / 61.5 against 61.5; 256 tokens, four
// of 128: 48.3 / 60.3 against 48.3; 512 tokens, sixteen of 128: 141 / 173 against 141; larger ones are equal.
int gemm_bf16_rope_tile(const GemmLaunch& g, int dh) {
  const int forced = bf16_forced_tile();
  if (forced >= 0)
    return (forced == TILE_L && (dh == 64 || dh == 128)) || (dh == 64 && (forced == TILE_M2 || forced == TILE_M4)) ? forced : -1;
  if (dh != 64 && dh != 128) return -1;
  int best = TILE_L;
  for (int c : {TILE_M2, TILE_M4})
    if (dh == 64 && bf16_tile_cost(g, c) < bf16_tile_cost(g, best)) best = c;
  float least;
  bf16_best_tile(g, &least);
  return bf16_tile_cost(g, best) <= least + 6.f ? best : -1;
}
static hipError_t run_rope(GemmLaunch& g, hipStream_t s) {
  switch (g.tile) {
    case TILE_L: return run_bf16<CfgL8, true, true, EPI_ROPE, PipeL, false>(g, s);
    case TILE_M2: return run_bf16<CfgM, true, true, EPI_ROPE, PipeM2>(g, s);
    case TILE_M4: return run_bf16<CfgM8, true, true, EPI_ROPE, PipeM4>(g, s);
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
  if (e == hipSuccess) e = Bf16Kernel<CfgL8, true, true, EPI_ROPE, PipeL, false>::prepare();
  if (e == hipSuccess) e = Bf16Kernel<CfgM, true, true, EPI_ROPE, PipeM2, true>::prepare();
  if (e == hipSuccess) e = Bf16Kernel<CfgM8, true, true, EPI_ROPE, PipeM4, true>::prepare();
  return e;
}
}  // namespace mecefo
