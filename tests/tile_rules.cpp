// What the planning functions choose, on the host.
//   tile_rules rope        every forward [b x d] with heads of 64 and 128: "b d dh configuration, modelled time of the shortest
//                          launch that rotates, of that configuration, of the best whole tiles" for Q, K and V
//   tile_rules cost EPI AKC BKC NPROB M N K F32     "modelled time on the 192-row tile, on 256 x 256 tiles, what cutting up
//                          their last round saves, the configuration taken" of a launch of NPROB equal products
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include "gemm_bf16_launch.hip.h"

using namespace mecefo;

static GemmLaunch launch(int epi, bool akc, bool bkc, int nprob, int M, int N, int K) {
  GemmLaunch g;
  memset(&g, 0, sizeof(g));
  g.a_kcontig = akc; g.b_kcontig = bkc; g.bf16 = true;
  g.epi = epi;
  g.nprob = nprob;
  for (int i = 0; i < nprob; ++i) {
    GemmProblem& p = g.p[i];
    p.M = M; p.N = N; p.K = K; p.nseg = 1;
  }
  return g;
}

int main(int argc, char** argv) {
  if (argc == 10 && !strcmp(argv[1], "cost")) {
    int v[8];
    for (int i = 0; i < 8; ++i) v[i] = atoi(argv[2 + i]);
    GemmLaunch g = launch(v[0], v[1], v[2], v[3], v[4], v[5], v[6]);
    g.out_f32 = v[7];
    printf("%.2f %.2f %.2f %d\n", bf16_tile_cost(g, TILE_K), bf16_tile_cost(g, TILE_L), bf16_tail(g).saved, bf16_best_tile(g));
    return 0;
  }
  if (argc != 2 || strcmp(argv[1], "rope")) return 1;
  for (int dh = 64; dh <= 128; dh += 64)
    for (int b = 256; b <= 8192; b += 256)
      for (int d = 512; d <= 4096; d += 128) {
        const GemmLaunch plain = launch(EPI_STORE, true, true, 3, b, d, d), rot = launch(EPI_ROPE, true, true, 3, b, d, d);
        const int c = gemm_bf16_rope_tile(plain, dh);
        float least, best = bf16_tile_cost(rot, TILE_L);
        bf16_best_tile(rot, &least);
        if (dh == 64) best = fminf(best, fminf(bf16_tile_cost(rot, TILE_M2), bf16_tile_cost(rot, TILE_M4)));
        printf("%d %d %d %d %.2f %.2f %.2f\n", b, d, dh, c, best, c < 0 ? best : bf16_tile_cost(rot, c), least);
      }
  return 0;
}
