// Host check of the store rule: one line where two buffers fill the last-level
// cache, whatever the element type, and one below which they fit the L2s.
#include "lattice.h"
#include <cstdio>
int main() {
  const size_t M = (size_t)1 << 20;
  int fails = 0;
  for (size_t mib : {23, 64, 119, 121, 127, 128}) fails += lbm::stores_past_caches(mib * M);
  for (size_t b : {M, 16 * M, 23 * M - 1, 128 * M + 1, 130 * M, 4096 * M}) fails += !lbm::stores_past_caches(b);
  printf("fails %d\n", fails);
  return fails != 0;
}
