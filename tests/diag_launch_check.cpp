// Host check of the diagnostics' launch: fewer than 2^32 threads for every grid
// that lbm_create takes, and the waves that the kernel's LDS is sized for.
#include "observe.h"
#include <cstdio>
using namespace lbm;
int main() {
  long fails = 0;
  for (int nx : {1, 64, 65, 256, 1024})
    for (int ny : {1, 2, 3, 5, 8, 64})
      for (int64_t nz : {1, 2, 16, 128, 100000, 8388607, 8388608, 20000000, 67108863}) {
        if (nx * ny * nz >= ((int64_t)1 << 31)) continue;
        const Grid g{nx, ny, (int)nz, nx * ny * nz, xblocks(nx)};
        const int t = diag_threads(g);
        const int64_t least = (int64_t)g.nxb * nz * 64;
        const bool fits = least < ((int64_t)1 << 32);
        if (t < 64 || t > kDiagThreads || t % 64 || (fits && (int64_t)g.nxb * nz * t >= ((int64_t)1 << 32)) ||
            (least * 8 < ((int64_t)1 << 32) && t != 64 * (ny >= 5 ? 8 : (ny >= 3 ? 4 : ny)))) {
          ++fails;
          printf("%d x %d x %lld: %d threads\n", nx, ny, (long long)nz, t);
        }
      }
  printf("fails %ld\n", fails);
  return fails != 0;
}
