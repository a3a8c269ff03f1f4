// Checks the block plans (lbm_plan.h) of FP32 lattices beyond the last-level cache
// against measured times: launches of two steps, which wait for HBM there (60.6 us a
// step at 2451^2, 102.5 at 3242^2), are not chosen, and the modelled time is within a
// tenth of the measured one.  Prints the number of sizes; exits 1 on a failure.
#include <cstdio>

#include "lbm_plan.h"

using namespace lbm;

struct Measured {
  int nx, ny;
  double us;  // a step, by launches of three steps
};

static const Measured kMeasured[] = {{1933, 1933, 30.1}, {2024, 2024, 35.0}, {2234, 2234, 42.4}, {2388, 2388, 48.5},
                                     {2451, 2451, 51.3}, {2556, 2556, 55.4}, {2689, 2689, 61.0}, {2752, 2752, 63.1},
                                     {3242, 3242, 87.7}, {3000, 3000, 76.0}, {3750, 1000, 30.3}, {5011, 1000, 43.4},
                                     {8018, 1000, 67.8}};

int main() {
  for (const Measured& m : kMeasured) {
    double us = 0.0;
    const BlockPlan p = plan_lattice(m.nx, m.ny, 4, 256, kBlockMinSteps, kBlockMaxSteps, &us);
    if (p.k < 3 || us < 0.9 * m.us || us > 1.1 * m.us) {
      std::printf("%d x %d: %d steps a launch, %.1f us a step, measured %.1f\n", m.nx, m.ny, p.k, us, m.us);
      return 1;
    }
  }
  std::printf("%zu sizes, 0 failures\n", sizeof kMeasured / sizeof *kMeasured);
  return 0;
}
