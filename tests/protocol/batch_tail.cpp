// Checks what ends a call on a batch in blocks (lbm_plan.h): launches add up to the steps
// for every count, the counted launches are those that run, and where the blocks and
// the tiles were measured and differ by more than a twelfth, the faster one runs.
// Prints the number of batches; exits 1 on a failure.
#include <cstdio>
#include <cstdlib>

#include "lbm_plan.h"

using namespace lbm;

// us of a call of one and of two steps, by blocks and by tiles
struct Measured {
  int es, n, nx, ny;
  double block1, tile1, block2, tile2;
};

static const Measured kMeasured[] = {
    {4, 1000, 64, 64, 78.7, 117.0, 97.0, 180.0},    {4, 8, 1024, 1024, 139.7, 129.2, 166.6, 157.8},
    {4, 16, 1024, 1024, 264.2, 248.4, 319.8, 298.2}, {4, 1, 2048, 2048, 77.4, 67.1, 92.4, 89.0},
    {4, 1, 3000, 3000, 154.8, 145.4, 181.4, 168.8}, {4, 2, 4096, 4096, 549.7, 462.4, 642.2, 541.0},
    {4, 100, 30, 1000, 48.4, 126.4, 58.0, 240.2},   {8, 1000, 64, 64, 134.9, 232.6, 176.6, 393.8},
    {8, 4, 1024, 1024, 135.8, 127.3, 177.2, 183.0}, {8, 4, 2048, 2048, 512.3, 469.1, 645.2, 579.6},
    {8, 1, 3000, 3000, 269.4, 273.4, 372.0, 325.2}, {8, 1, 4096, 4096, 497.4, 461.0, 667.4, 562.8},
    {8, 100, 30, 1000, 138.4, 296.1, 144.8, 569.8},
};

static int batches = 0;

static void fail(const char* what, int es, int n, int nx, int ny) {
  std::printf("%s: element %d, %d domains of %d x %d\n", what, es, n, nx, ny);
  std::exit(1);
}

static BatchBlocks check(int es, int n, int nx, int ny) {
  ++batches;
  const BatchBlocks p = plan_batch(std::vector<DomainSize>(n, DomainSize{nx, ny}), es, 256);
  if (p.k < 1 || p.whole) return p;
  for (int steps = 1; steps <= 100; ++steps) {
    int left = steps, launches = 0;
    for (; left > 0; ++launches) {
      const BatchLaunch q = p.next(left);
      if (q.steps < 1 || q.steps > left || q.steps > (q.tiles ? 2 : p.k)) fail("launch", es, n, nx, ny);
      left -= q.steps;
    }
    if (launches != p.launches(steps)) fail("launches", es, n, nx, ny);
  }
  return p;
}

int main() {
  for (const Measured& m : kMeasured) {
    const BatchBlocks p = check(m.es, m.n, m.nx, m.ny);
    const double one = p.next(1).tiles ? m.tile1 : m.block1;
    const double two = p.next(2).steps == 2 ? (p.next(2).tiles ? m.tile2 : m.block2) : 1e300;
    if (one > 13.0 / 12.0 * std::min(m.block1, m.tile1)) fail("one step", m.es, m.n, m.nx, m.ny);
    if (two > 13.0 / 12.0 * std::min(m.block2, m.tile2)) fail("two steps", m.es, m.n, m.nx, m.ny);
  }
  for (int es : {4, 8})
    for (int n : {1, 7, 60, 500})
      for (int nx : {3, 50, 200, 700})
        for (int ny : {4, 100, 333}) check(es, n, nx, ny);
  std::printf("%d batches, 0 failures\n", batches);
  return 0;
}
