// Host check of the rule that takes steps two at a time: grids whose pairs were
// measured slower than single steps stay single, and those that gain by 15 % and
// more stay paired (256 CUs; the gains are those of 40 steps).
#include "twostep.h"
#include <cstdio>
using namespace lbm;
struct Case {
  int nx, ny, nz, qt, bytes;
  Rates rates;
  double gain;  // single / paired
};
int main() {
  constexpr Rates U = Rates::kUnit, P = Rates::kParametrised, G = Rates::kGiven;
  const Case cases[] = {
      // slower in pairs; the rule without the collision took them
      {962, 19, 90, 34, 4, G, 0.922}, {1056, 29, 46, 34, 4, G, 0.890}, {372, 27, 67, 34, 4, G, 0.956},
      {696, 8, 61, 34, 4, G, 0.824}, {696, 8, 61, 34, 4, U, 0.967}, {655, 27, 93, 54, 4, G, 0.857},
      {908, 20, 73, 54, 4, G, 0.868}, {511, 25, 52, 54, 4, G, 0.856}, {494, 22, 53, 54, 4, P, 0.919},
      {372, 29, 32, 34, 8, G, 0.893}, {457, 25, 23, 34, 8, G, 0.848}, {457, 25, 23, 34, 8, P, 0.965},
      {335, 40, 25, 25, 8, U, 0.973}, {120, 59, 37, 25, 8, U, 0.916}, {254, 23, 44, 25, 8, U, 0.879},
      // slower in pairs, refused before as well
      {277, 23, 41, 34, 4, U, 0.913}, {389, 11, 106, 54, 4, U, 0.957}, {144, 38, 41, 34, 8, U, 0.892},
      {914, 71, 31, 54, 4, P, 0.966}, {951, 17, 123, 54, 4, G, 0.811},
      // faster in pairs
      {1024, 64, 128, 34, 4, U, 1.53}, {1024, 64, 128, 34, 4, G, 1.22}, {1024, 64, 128, 54, 4, G, 1.31},
      {1024, 64, 128, 54, 4, P, 1.52}, {1024, 64, 128, 34, 8, G, 1.37}, {1024, 64, 128, 25, 8, U, 1.35},
      {512, 32, 64, 34, 4, G, 1.20}, {512, 32, 64, 34, 4, P, 1.37}, {505, 22, 56, 34, 4, U, 1.18},
      {311, 33, 57, 34, 4, P, 1.20}, {738, 24, 36, 54, 4, U, 1.20}, {104, 60, 123, 54, 4, U, 1.25},
      {349, 46, 33, 34, 8, U, 1.34}, {349, 46, 33, 34, 8, G, 1.24}, {442, 26, 49, 34, 8, G, 1.21},
      {100, 71, 125, 25, 8, U, 1.24}, {286, 18, 122, 25, 8, U, 1.18}, {552, 21, 95, 34, 4, P, 1.46}, {552, 21, 95, 34, 4, G, 1.25}};
  int fails = 0;
  for (const Case& c : cases) {
    const Grid g{c.nx, c.ny, c.nz, (int64_t)c.nx * c.ny * c.nz, xblocks(c.nx)};
    const size_t state = (size_t)g.nxb * kXB * c.ny * c.nz * c.qt * c.bytes;
    if (two_step_pays(g, c.qt, c.bytes, 256, c.rates, state) != (c.gain > 1)) {
      ++fails;
      printf("%d x %d x %d, %d populations of %d bytes, rates %d\n", c.nx, c.ny, c.nz, c.qt, c.bytes, (int)c.rates);
    }
  }
  printf("fails %d\n", fails);
  return fails != 0;
}
