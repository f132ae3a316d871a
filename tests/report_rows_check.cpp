// Host check of the reporting kernels' pulls on rows of any length: the pointer
// at the tile's first x-block plus the segment plus the lane's offset is the
// element that the reference pull names, up to the longest rows a grid may have.
#include "lattice.h"
#include <cstdio>
using namespace lbm;
static long fails = 0;
template <class LF, class LS>
void check(int nx, int bdim) {
  constexpr int QT = LF::Q + LS::Q;
  const Grid g{nx, 1, 3, (int64_t)nx * 3, xblocks(nx)};
  const int tiles = (nx + bdim - 1) / bdim;
  const char* none = nullptr;  // one byte per element: addresses only, never read
  for (int tile : {0, 1, tiles / 3, tiles / 2, tiles - 2, tiles - 1}) {
    if (tile < 0 || tile >= tiles) continue;
    const int x0 = tile * bdim, xb0 = x0 >> kXBShift;
    const int64_t at = (int64_t)xb0 * (QT * kXB);
    for (int tid = 0; tid < bdim; ++tid) {
      const auto t = tile_lanes<QT, 1>(g, x0, tid, bdim, xb0);
      if (t.x[0] >= nx) continue;
      for (int z = 0; z < 3; ++z) {
        auto pull = [&](auto lat, auto base_c) {
          using L = decltype(lat);
          constexpr int base = decltype(base_c)::value;
          static_for<0, L::Q>([&](auto qc) {
            constexpr int q = decltype(qc)::value;
            bool zw;
            int64_t e = at + pull_segment<L, q, base, QT>(g, 0, z, zw) + pull_lane<L, q, QT, 1>(t, 0, zw);
            if (x_wall<L, q>(g, t.x[0], zw)) e = at + bounce_segment<L, q, base, QT>(g, 0, z) + t.own[0];
            if (e != pull_ptr<L, q, QT>(none, g, base, t.x[0], 0, z) - none && ++fails < 10)
              printf("nx %d x %d z %d pop %d: element %lld\n", nx, t.x[0], z, base + q, (long long)e);
          });
        };
        pull(LF{}, std::integral_constant<int, 0>{});
        pull(LS{}, std::integral_constant<int, LF::Q>{});
      }
    }
  }
}
int main() {
  for (int nx : {1, 64, 65, 300, 39768215, 39768300, 63161284, 100000001, 600000000})
    for (int bdim : {64, 128, 256}) {
      check<Q27, Q7>(nx, bdim);
      check<Q19, Q6>(nx, bdim);
      check<Q27, Q27>(nx, bdim);
    }
  printf("fails %ld\n", fails);
  return fails != 0;
}
