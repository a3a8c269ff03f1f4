// Checks the search of the block plans (lbm_plan.h), which skips what cannot be the
// best, against one that tries every division in every shape: the same plans for many
// sizes.  Prints the number of plans; exits 1 on a failure.
#include <cstdio>

#include "lbm_plan.h"

using namespace lbm;

static BlockPlan exhaustive(int nx, int rows, int es, int cus, int min_k, int max_k, double* us) {
  const BlockCost c = block_cost(es);
  const bool far = block_beyond_cache(es, (long long)nx * rows);
  if (far) min_k = std::max(min_k, 3);
  BlockPlan best{};
  *us = 1e300;
  for (BlockShape s : kBlockShapes) {
    const int r = block_resident(es, s);
    if (!block_shape_built(es, s) || (far && r < 2)) continue;
    for (int k = max_k; k >= min_k; --k)
      for_block_widths(nx, [&](int ntx) {
        const int fewest = block_rows(nx, rows, ntx, k, s.threads * s.cells), halo = 2 * (2 * k - 1);
        for (int round = 0; fewest > 0 && round <= 4; ++round) {
          const int nty = round == 0 ? fewest : std::min(rows, round * cus / ntx);
          if (nty < fewest) continue;
          const int w = (nx + ntx - 1) / ntx, h = (rows + nty - 1) / nty;
          const double moved = (double)(w + halo) * (h + halo) + (double)w * h, q = (ntx * nty + cus - 1) / cus;
          const double t = std::max(block_launch_time(c, k, q, block_work(c, w + halo, h + halo, k), moved, r),
                                    hbm_time(es, (double)nx * rows, ntx * nty * moved)) / k;
          if (t >= *us) continue;
          *us = t;
          best = block_plan(nx, rows, k, ntx, nty, s);
        }
      });
  }
  return best;
}

int main() {
  int plans = 0;
  for (int es : {4, 8})
    for (int cus : {256, 64})
      for (int min_k : {kBlockMinSteps, 2})
        for (int nx : {3, 5, 31, 64, 100, 200, 333, 512, 777, 1000, 1448, 2451, 5011})
          for (int rows : {3, 4, 37, 64, 120, 200, 513, 1000, 1448, 2389}) {
            const int max_k = min_k == 2 && cus == 64 ? 2 : kBlockMaxSteps;
            double want = 0.0, got = 0.0;
            const BlockPlan a = exhaustive(nx, rows, es, cus, min_k, max_k, &want);
            const BlockPlan b = plan_lattice(nx, rows, es, cus, min_k, max_k, &got);
            ++plans;
            if (a.k != b.k || a.ntx != b.ntx || a.nty != b.nty || a.threads != b.threads || a.cells != b.cells || want != got) {
              std::printf("%d x %d element %d: k %d, %d x %d blocks of %d x %d for k %d, %d x %d of %d x %d\n", nx, rows, es,
                          b.k, b.ntx, b.nty, b.threads, b.cells, a.k, a.ntx, a.nty, a.threads, a.cells);
              return 1;
            }
          }
  std::printf("%d plans, 0 failures\n", plans);
  return 0;
}
