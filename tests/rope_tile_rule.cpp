// For every forward [b x d] with heads of 64 and 128: the launch that goes out for Q, K and V, by the model of the tiles.
// Prints "b d dh configuration, its time, the time of the best tiles without rotation" for the sizes of the sweep.
#include <stdio.h>
#include <string.h>

#include "gemm_bf16_launch.hip.h"

using namespace mecefo;

static GemmLaunch qkv(int b, int d, int epi) {
  GemmLaunch g;
  memset(&g, 0, sizeof(g));
  g.a_kcontig = g.b_kcontig = g.bf16 = true;
  g.epi = epi;
  g.nprob = 3;
  for (int i = 0; i < 3; ++i) {
    GemmProblem& p = g.p[i];
    p.M = b; p.N = p.K = d; p.lda = p.ldb = p.ldc = d; p.nseg = 1;
  }
  return g;
}

int main() {
  for (int dh = 64; dh <= 128; dh += 64)
    for (int b = 256; b <= 8192; b += 256)
      for (int d = 512; d <= 4096; d += 128) {
        const GemmLaunch plain = qkv(b, d, EPI_STORE), rot = qkv(b, d, EPI_ROPE);
        const int c = gemm_bf16_rope_tile(plain, dh);
        float least;
        bf16_best_tile(plain, &least);
        printf("%d %d %d %d %.2f %.2f\n", b, d, dh, c, c < 0 ? least : bf16_tile_cost(rot, c), least);
      }
  return 0;
}
