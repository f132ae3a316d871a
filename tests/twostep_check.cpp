// Host check of the two-step kernel's addressing: every tile, wave and lane of
// a launch, with populations replaced by labels. The first step's result at
// (population, node) is labelled with that pair; what the second step reads
// from LDS must be the label that the reference pull (pull_ptr) names, in the
// kernel's order of phases, and every global and LDS index must be in bounds.
#include "twostep.h"
#include <cstdio>
#include <vector>
using namespace lbm;
static long fails = 0;
static void bad(const char* what, int nx, int ny, int nz, int x, int y, int z, int a) {
  if (++fails < 10) printf("%s grid %d %d %d node %d %d %d pop %d\n", what, nx, ny, nz, x, y, z, a);
}
template <class LF, class LS, int TY>
void check(int nx, int ny, int nz, int zc) {
  using P = Pops<LF, LS>;
  constexpr int QT = P::Q;
  Grid g{nx, ny, nz, (int64_t)nx * ny * nz, xblocks(nx)};
  TwoStep s;
  s.ntx = g.nxb;
  s.nty = (ny + TY - 1) / TY;
  s.zc = zc;
  s.nblocks = s.ntx * s.nty * ((nz + zc - 1) / zc);
  const int64_t plane = (int64_t)ny * g.nxb * (QT * kXB), total = plane * nz;
  const int nlds = P::kSlots * TY * kPitch;
  std::vector<char> stored(total, 0);
  const float* base0 = nullptr;
  auto ref = [&](int a, int x, int y, int z) {  // element of the pull of a at (x, y, z)
    int64_t e = -1;
    static_for<0, LF::Q>([&](auto qc) {
      constexpr int q = decltype(qc)::value;
      if (a == q) e = pull_ptr<LF, q, QT>(base0, g, 0, x, y, z) - base0;
    });
    static_for<0, LS::Q>([&](auto qc) {
      constexpr int q = decltype(qc)::value;
      if (a == LF::Q + q) e = pull_ptr<LS, q, QT>(base0, g, LF::Q, x, y, z) - base0;
    });
    return e;
  };
  for (int b = 0; b < s.nblocks; ++b) {
    const Tile tile = tile_of(g, s, TY, b);
    if (tile.xb < 0 || tile.xb >= g.nxb || tile.y0 < 0 || tile.y0 >= ny || tile.rows < 1 ||
        tile.y0 + tile.rows > ny || tile.z0 < 0 || tile.z0 >= tile.z1 || tile.z1 > nz)
      bad("tile", nx, ny, nz, tile.xb, tile.y0, tile.z0, 0);
    std::vector<int64_t> lds(nlds, -1);
    const int ks = tile.z0 > 0 ? tile.z0 - 1 : 0;
    for (int k = ks; k <= tile.z1; ++k) {
      // the three phases of an iteration, each over every lane of the block
      for (int phase = 0; phase < 3; ++phase)
        for (int w = 0; w < TY + 3; ++w)
          for (int lane = 0; lane < 64; ++lane) {
            const Lane l = lane_of(g, tile, TY, w, lane);
            const int at = lds_lane(l, lane);
            if (l.x < 0 || l.x >= nx || l.y < 0 || l.y >= ny) bad("lane", nx, ny, nz, l.x, l.y, k, w);
            auto put = [&](auto ac, int i) {
              constexpr int a = decltype(ac)::value;
              if (i < 0 || i >= nlds) return bad("lds", nx, ny, nz, l.x, l.y, k, a);
              lds[i] = elem_index<QT>(g, a, (int64_t)k * ny + l.y, l.x);
            };
            if (phase == 0 && k < nz) {
              uint32_t off[3][3];
              plane_offsets<QT, float>(g, l.x, l.y, off);
              static_for<0, QT>([&](auto ac) {  // the first step's pull
                constexpr int a = decltype(ac)::value;
                constexpr int cx = P::cx(a), cy = P::cy(a), cz = P::cz(a);
                int pz = k - cz;
                if (pz < 0 || pz >= nz) pz = k;
                int64_t e = pz * plane + a * kXB + off[cy + 1][cx + 1] / 4;
                if (e < 0 || e >= total) bad("load", nx, ny, nz, l.x, l.y, k, a);
                const bool wall = (cz == 1 && k == 0) || (cz == -1 && k == nz - 1) ||
                                  (cx == 1 && l.x == 0) || (cx == -1 && l.x == nx - 1);
                if (wall) e = k * plane + P::opposite(a) * kXB + off[1][1] / 4;
                if (e < 0 || e >= total) bad("fix-up", nx, ny, nz, l.x, l.y, k, a);
                if (l.active && e != ref(a, l.x, l.y, k)) bad("pull", nx, ny, nz, l.x, l.y, k, a);
              });
              if (l.active) push_class<P, TY, -1>(l, w < TY + 2, w - 1, tile.rows, at + class_base<P, TY>(-1, k - 1), at, put);
            } else if (phase == 1 && k > tile.z0 && w < tile.rows) {
              const int x = tile.xb * kXB + lane, y = tile.y0 + w, z = k - 1;
              static_for<0, QT>([&](auto ac) {  // the second step's pull and store
                constexpr int a = decltype(ac)::value;
                const int i = w * kPitch + 1 + lane + class_base<P, TY>(P::cz(a), z) + class_offset<P, TY>(a, 0, 0);
                if (i < 0 || i >= nlds) return bad("lds read", nx, ny, nz, x, y, z, a);
                if (x >= nx) return;
                if (lds[i] != ref(a, x, y, z)) bad("second pull", nx, ny, nz, x, y, z, a);
                const int64_t e = z * plane + ((int64_t)y * g.nxb + tile.xb) * (QT * kXB) + a * kXB + lane;
                if (e < 0 || e >= total || e != elem_index<QT>(g, a, (int64_t)z * ny + y, x)) return bad("store", nx, ny, nz, x, y, z, a);
                if (stored[e]++) bad("stored twice", nx, ny, nz, x, y, z, a);
              });
            } else if (phase == 2 && k < nz && l.active) {
              push_class<P, TY, 0>(l, w < TY + 2, w - 1, tile.rows, at + class_base<P, TY>(0, k), at, put);
              push_class<P, TY, 1>(l, w < TY + 2, w - 1, tile.rows, at + class_base<P, TY>(1, k + 1), at, put);
              if (w < TY + 2 && (unsigned)(w - 1) < (unsigned)tile.rows)
                { const int base[3] = {at + class_base<P, TY>(-1, k), at + class_base<P, TY>(0, k), at + class_base<P, TY>(1, k)}; push_bounce<P, TY>(g, l, base, k, put); }
            }
          }
    }
  }
  int64_t n = 0;
  for (char c : stored) n += c;
  if (n != g.n * QT) bad("nodes not stored", nx, ny, nz, 0, 0, 0, (int)(g.n * QT - n));
}
template <class LF, class LS, int TY>
void grids() {
  for (int nx : {1, 2, 63, 64, 65, 66, 127, 129})
    for (int ny : {1, 2, TY - 1, TY, TY + 1, 2 * TY + 1})
      for (int nz : {1, 2, 3, 5}) {
        if (nx > 66 && ny > TY) continue;
        check<LF, LS, TY>(nx, ny, nz, nz);
        if (nz > 1) check<LF, LS, TY>(nx, ny, nz, nz / 2);
        if (nz > 2) check<LF, LS, TY>(nx, ny, nz, 1);
      }
}
// the planned split covers every plane of every tile once
static void plans() {
  for (int nx : {1, 64, 65, 1024})
    for (int ny : {1, 7, 8, 64})
      for (int nz : {1, 2, 31, 128})
        for (int cus : {1, 64, 256}) {
          Grid g{nx, ny, nz, (int64_t)nx * ny * nz, xblocks(nx)};
          TwoStep s;
          two_step_plan(g, 8, cus, s);
          int64_t planes = 0;
          for (int b = 0; b < s.nblocks; ++b) {
            const Tile t = tile_of(g, s, 8, b);
            if (t.z0 < 0 || t.z1 <= t.z0 || t.z1 > nz || t.xb >= g.nxb) bad("plan", nx, ny, nz, t.xb, t.y0, t.z0, cus);
            planes += (int64_t)(t.z1 - t.z0) * t.rows;
          }
          if (planes != (int64_t)g.nxb * ny * nz) bad("plan cover", nx, ny, nz, 0, 0, 0, cus);
        }
}
int main() {
  plans();
  grids<Q27, Q7, 8>();
  grids<Q27, Q7, 3>();
  grids<Q19, Q6, 8>();
  grids<Q27, Q27, 4>();
  printf("fails %ld\n", fails);
  return fails != 0;
}
