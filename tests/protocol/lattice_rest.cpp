// Checks what ends a call on a lattice in blocks (lbm_plan.h) against measured times:
// wherever the blocks and the marching tiles differ by more than a twelfth, the
// faster one runs.  Prints the number of sizes; exits 1 on a failure.
#include <cstdio>
#include <cstdlib>

#include "lbm_plan.h"

using namespace lbm;

// us a call of one and of two steps, by blocks and by tiles; lanes of a row of strips of either shape
struct Measured {
  int es, nx, ny, lanes1, lanes2;
  double block1, tile1, block2, tile2;
};

static const Measured kMeasured[] = {
    {4, 700, 700, 768, 768, 8.8, 13.4, 12.9, 22.6},       {4, 886, 886, 1024, 1024, 12.9, 14.7, 17.4, 24.3},
    {4, 1000, 1000, 1024, 1152, 16.1, 15.6, 21.3, 28.4},  {4, 1254, 1254, 1280, 1408, 22.5, 21.9, 29.9, 32.5},
    {4, 1448, 1448, 1536, 1536, 28.8, 27.4, 38.6, 38.9},  {4, 2048, 2048, 2048, 2176, 69.4, 57.7, 85.6, 78},
    {4, 1700, 1700, 1792, 1792, 38.4, 36.1, 50.1, 53.8},
    {4, 2600, 2600, 2816, 2816, 120.1, 108.1, 136.9, 131.9}, {4, 3400, 3400, 3584, 3584, 192.3, 190.3, 231.2, 203.1},
    {4, 4096, 400, 4096, 4352, 25.3, 22.4, 32.2, 32.4},   {4, 500, 4000, 512, 640, 26.9, 24.3, 35.7, 45.3},
    {4, 128, 8000, 128, 256, 16, 15.5, 20.9, 40.9},     {4, 300, 5000, 512, 384, 22.1, 22.9, 28.1, 33},
    {8, 700, 700, 768, 768, 14, 19.5, 18.6, 28.9},      {8, 1000, 1000, 1024, 1024, 25.9, 24.5, 32.2, 34.8},
    {8, 1130, 1130, 1280, 1280, 31.2, 31.7, 42.2, 43.1},
    {8, 1254, 1254, 1280, 1536, 37.1, 42.2, 51.9, 51.2},  {8, 1448, 1448, 1536, 1536, 68.5, 65.8, 84.6, 78.8},
    {8, 2048, 2048, 2048, 2304, 131.9, 117.7, 164.7, 144.5}, {8, 2600, 2600, 2816, 2816, 209.7, 202.3, 254.9, 225.2},
    {8, 4096, 400, 4096, 4352, 41.5, 43.1, 54.5, 50.2},   {8, 500, 4000, 512, 512, 57.5, 61, 78.2, 73.5},
    {8, 300, 5000, 512, 512, 37.1, 40.7, 48.2, 62.2},     {8, 128, 8000, 128, 256, 25.2, 24.6, 33.3, 66.7},
};

int main() {
  for (const Measured& m : kMeasured) {
    const LatticeRest r = lattice_rest(m.es, m.nx, m.ny, m.lanes1, m.lanes2);
    const double one = r.one ? m.tile1 : m.block1, two = r.two ? m.tile2 : m.block2;
    if (one > 13.0 / 12.0 * std::min(m.block1, m.tile1) || two > 13.0 / 12.0 * std::min(m.block2, m.tile2)) {
      std::printf("element %d, %d x %d: one step by %s, two by %s\n", m.es, m.nx, m.ny, r.one ? "tiles" : "blocks",
                  r.two ? "tiles" : "blocks");
      return 1;
    }
  }
  // the steps of a call always add up, and no launch takes more than k
  for (int k = 1; k <= kBlockMaxSteps; ++k)
    for (bool two : {false, true})
      for (int n = 1; n <= 40; ++n) {
        int left = n;
        while (left > 0) {
          const int s = lattice_next_steps(left, k, {two, two});
          if (s < 1 || s > k || s > left) return 1;
          left -= s;
        }
      }
  std::printf("%zu sizes, 0 failures\n", sizeof kMeasured / sizeof *kMeasured);
  return 0;
}
