// Driver for tests/test_batch_places.py: records of a batch, one of them damaged, counted by BatchPlaces.  argv: the damaged
// place's expert and slot.  Prints the damaged record's index (-1: none), the misses and the sum of the counts.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "batch_places.h"

int main(int argc, char **argv) {
  if (argc != 3) return 2;
  constexpr int kTokens = 5, kTopK = 3, kExperts = 9, kCapacity = 6;
  std::vector<moe_route_out_t> rec(kTokens, moe_route_out_t{});
  for (int t = 0; t < kTokens; ++t)
    for (int k = 0; k < kTopK; ++k) {
      rec[t].sel_expert[k] = (t + k) % kExperts;
      rec[t].sel_slot[k] = (t + k) % kCapacity;
      rec[t].miss[k] = t == 1 && k == 2;
    }
  rec[3].sel_expert[1] = std::atoi(argv[1]);
  rec[3].sel_slot[1] = std::atoi(argv[2]);
  moe::BatchPlaces p;
  const moe_route_out_t *bad = p.count(rec.data(), kTokens, kTopK, kExperts, kCapacity);
  int sum = 0;
  for (int n : p.of_slot) sum += n;
  std::printf("%d %d %d\n", bad ? (int)(bad - rec.data()) : -1, p.misses, sum);
  return 0;
}
