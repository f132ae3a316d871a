// The host check of the two-step kernel's addressing (twostep_check.cpp) on the
// tile shapes that the library launches, by element type: rows per tile, LDS,
// byte offsets inside a plane and the split into chunks.
#define main other_shapes
#include "twostep_check.cpp"
#undef main

template <class LF, class LS, typename T>
static void shipped() {
  using P = Pops<LF, LS>;
  constexpr int TY = two_step_rows((int)sizeof(T));
  static_assert(P::kSlots * TY * kPitch * sizeof(T) <= 160 * 1024, "LDS of one block");
  grids<LF, LS, TY>();
  for (int nx : {1, 64, 65, 1000})
    for (int ny : {1, 2, 5, 64}) {
      const Grid g{nx, ny, 2, (int64_t)nx * ny * 2, xblocks(nx)};
      for (int y = 0; y < ny; ++y)
        for (int x : {0, 1, 62, 63, 64, nx - 2, nx - 1}) {
          if (x < 0 || x >= nx) continue;
          uint32_t off[3][3];
          plane_offsets<P::Q, T>(g, x, y, off);
          for (int cy = -1; cy <= 1; ++cy)
            for (int cx = -1; cx <= 1; ++cx) {
              const int xs = x - cx < 0 || x - cx >= nx ? x : x - cx, ys = (y - cy + ny) % ny;
              if (off[cy + 1][cx + 1] != elem_index<P::Q>(g, 0, ys, xs) * (int64_t)sizeof(T))
                bad("offset", nx, ny, 2, x, y, 0, 0);
            }
        }
    }
}
static void splits(int ty) {
  for (int nx : {1, 65, 1024})
    for (int ny : {1, 4, 5, 6, 8, 9, 64})
      for (int nz : {1, 2, 31, 128})
        for (int cus : {1, 64, 256}) {
          const Grid g{nx, ny, nz, (int64_t)nx * ny * nz, xblocks(nx)};
          TwoStep s;
          two_step_plan(g, ty, cus, s);
          std::vector<char> done((size_t)g.nxb * ny * nz, 0);
          for (int b = 0; b < s.nblocks; ++b) {
            const Tile t = tile_of(g, s, ty, b);
            for (int y = t.y0; y < t.y0 + t.rows; ++y)
              for (int z = t.z0; z < t.z1; ++z) {
                if (t.xb < 0 || t.xb >= g.nxb || y < 0 || y >= ny || z < 0 || z >= nz ||
                    done[((size_t)z * ny + y) * g.nxb + t.xb]++)
                  bad("split", nx, ny, nz, t.xb, y, z, cus);
              }
          }
          for (char c : done)
            if (!c) bad("split misses", nx, ny, nz, 0, 0, 0, cus);
        }
}
int main() {
  splits(two_step_rows(4));
  splits(two_step_rows(8));
  shipped<Q27, Q7, float>();
  shipped<Q27, Q7, double>();
  shipped<Q19, Q6, double>();
  shipped<Q27, Q27, float>();
  printf("fails %ld\n", fails);
  return fails != 0;
}
