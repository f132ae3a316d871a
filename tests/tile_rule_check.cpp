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
  // few waves: whole rows of two and four whose last wave is nearly empty
  for (int64_t rows : {20, 100, 150, 256}) {
    for (int nx : {65, 80, 96}) want(nx, rows, 1, 256, 128);
    for (int nx : {97, 112, 128}) want(nx, rows, 1, 256, 64);
  }
  for (int nx : {193, 208}) {
    want(nx, 72, 1, 256, 256);
    want(nx, 128, 1, 256, 256);
    want(nx, 64, 1, 256, 64);
    want(nx, 128, 1, 0, 64);
  }
  for (int nx : {209, 224, 225, 256}) want(nx, 100, 1, 256, 64);
  want(129, 150, 1, 256, 64);
  want(257, 90, 1, 256, 64);
  want(576, 496, 1, 256, 64);
  for (int nx = 1; nx <= 512; ++nx)
    for (int64_t rows : {1, 30, 70, 100, 128, 200, 256, 300, 470, 500, 600, 5000})
      for (int cus : {64, 256, 304}) {
        const int t = tile_threads(nx, rows, 1, cus), least = tile_threads(nx, rows, 1, 0);
        const int waves = (nx + 63) / 64;
        if (t % 64 || t < 64 || t > 256 || waves % (t / 64) || (nx + t - 1) / t > (nx + least - 1) / least)
          ++fails, printf("%d x %lld on %d: %d\n", nx, (long long)rows, cus, t);
      }
  printf("fails %d\n", fails);
  return fails != 0;
}
