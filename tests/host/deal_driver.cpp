// Driver for tests/test_deal.py: how a workgroup's list of records is dealt out to its wavefronts, printed for lists read from
// stdin (pairs "ns nr"): per wavefront  first_sh n_sh first_rt n_rt  for STEP = NW, then for STEP = 1.
#include <cstdio>

#include "deal.h"

constexpr int NW = 8;

int main() {
  int ns, nr;
  while (scanf("%d %d", &ns, &nr) == 2) {
    for (int w = 0; w < NW; ++w) {
      const moe::Deal d = moe::deal<NW, NW>(ns, nr, w);
      printf("%d %d %d %d ", d.first_sh, d.n_sh, d.first_rt, d.n_rt);
    }
    for (int w = 0; w < NW; ++w) {
      const moe::Deal d = moe::deal<NW, 1>(ns, nr, w);
      printf("%d %d %d %d ", d.first_sh, d.n_sh, d.first_rt, d.n_rt);
    }
    printf("\n");
  }
  return 0;
}
