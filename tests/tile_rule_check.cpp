// Host check of the row tiles' blocks: whole waves of a row, none past its end
// (rows of one to eight waves), whole rows of three waves only where they fill
// the CUs two deep, and never more blocks than the adjoint's workspace counts.
#include "lattice.h"
#include <cstdio>
using namespace lbm;
int main() {
  int fails = 0;
  const auto want = [&](int nx, int64_t rows, int npt, int cus, int threads) {
    const int t = tile_threads(nx, rows, npt, cus);
    if (t != threads) ++fails, printf("%d x %lld, %d per thread: %d for %d\n", nx, (long long)rows, npt, t, threads);
  };
  for (int nx : {129, 162, 192}) {
    for (int64_t rows : {436, 460, 496, 512}) want(nx, rows, 1, 256, 192);
    for (int64_t rows : {171, 256, 280, 360, 435, 513, 528, 640, 1024, 1536, 5000}) want(nx, rows, 1, 256, 64);
    want(nx, 496, 1, 0, 64);
  }
  want(384, 496, 2, 256, 64);
  want(128, 496, 1, 256, 128);
  want(256, 496, 1, 256, 256);
  want(256, 128, 1, 256, 64);
  want(576, 496, 1, 256, 64);
  for (int nx = 1; nx <= 512; ++nx)
    for (int64_t rows : {1, 100, 300, 470, 500, 600, 5000})
      for (int cus : {64, 256, 304}) {
        const int t = tile_threads(nx, rows, 1, cus), least = tile_threads(nx, rows, 1, 0);
        const int waves = (nx + 63) / 64;
        if (t % 64 || t < 64 || t > 256 || waves % (t / 64) || (nx + t - 1) / t > (nx + least - 1) / least)
          ++fails, printf("%d x %lld on %d: %d\n", nx, (long long)rows, cus, t);
      }
  printf("fails %d\n", fails);
  return fails != 0;
}
