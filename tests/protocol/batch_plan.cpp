// Checks the block plans of batches (lbm_plan.h) on the host: the plan of a batch is
// the same in any order of its domains, the time it claims is the sum over all of
// its blocks, and the steps and shape chosen from a sample of the sizes cost at
// most a quarter more than the best ones for the whole batch.  Prints the number of
// batches; exits 1 on a failure.
#include <cstdio>
#include <cstdlib>
#include <random>

#include "lbm_plan.h"

using namespace lbm;

using Batch = std::vector<DomainSize>;

static void fail(const char* what, const Batch& dom, int es, const BatchBlocks& p) {
  std::printf("%s: %zu domains from %d x %d, element %d, k %d, %d x %d cells, %.2f us\n", what, dom.size(), dom[0].nx,
              dom[0].ny, es, p.k, p.shape.threads, p.shape.cells, p.us_per_step);
  std::exit(1);
}

static double all_cells(const Batch& dom) {
  double n = 0.0;
  for (const auto& d : dom) n += (double)d.nx * d.ny;
  return n;
}

// Time a step of blocks of k steps, domain by domain; 0 if a domain does not fit.
static double time_of(const Batch& dom, int es, int k, BlockShape s, const std::vector<int>* ntx, const std::vector<int>* nty,
                      int finer) {
  const BlockCost c = block_cost(es);
  BatchLaunchCost sum{es, k, block_resident(es, s)};
  const int halo = 2 * (2 * k - 1);
  for (size_t d = 0; d < dom.size(); ++d) {
    BlockCut q;
    if (ntx) {
      q.ntx = (*ntx)[d];
      q.nty = (*nty)[d];
      const int w = (dom[d].nx + q.ntx - 1) / q.ntx, h = (dom[d].ny + q.nty - 1) / q.nty;
      q.work = q.ntx * q.nty * block_work(c, w + halo, h + halo, k);
      q.cells = (double)q.ntx * q.nty * ((w + halo) * (h + halo) + w * h);
    } else {
      q = cut_domain(c, dom[d], s, k, finer);
    }
    if (q.ntx == 0) return 0.0;
    sum.add(q, 1.0);
  }
  return sum.us(all_cells(dom), 256) / k;
}

static int batches = 0;

static void check(Batch dom, int es, unsigned seed) {
  ++batches;
  const BatchBlocks p = plan_batch(dom, es, 256);
  if (p.k < 1) fail("no plan", dom, es, p);
  if (p.whole) return;
  const double claimed = p.us_per_step, full = time_of(dom, es, p.k, p.shape, &p.ntx, &p.nty, 1);
  if (std::fabs(claimed / full - 1.0) > 1e-9) fail("claimed time", dom, es, p);
  double best = 1e300;
  const bool far = block_beyond_cache(es, (long long)all_cells(dom));
  for (BlockShape s : kBlockShapes) {
    if (!block_shape_built(es, s) || (far && block_resident(es, s) < 2)) continue;
    for (int k = far ? 3 : 2; k <= kBlockMaxSteps; ++k) {
      const double t = time_of(dom, es, k, s, nullptr, nullptr, 1);
      if (t > 0.0) best = std::min(best, t);
    }
  }
  if (claimed > 1.25 * best) fail("far from the best", dom, es, p);
  // any order of the domains
  std::vector<int> order(dom.size());
  for (size_t d = 0; d < dom.size(); ++d) order[d] = (int)d;
  std::mt19937 g(seed);
  for (int turn = 0; turn < 3; ++turn) {
    if (turn == 0)
      std::reverse(order.begin(), order.end());
    else
      std::shuffle(order.begin(), order.end(), g);
    Batch other;
    for (int d : order) other.push_back(dom[d]);
    const BatchBlocks q = plan_batch(other, es, 256);
    if (q.k != p.k || q.shape.threads != p.shape.threads || q.shape.cells != p.shape.cells ||
        q.us_per_step != p.us_per_step || q.tiles_us_per_step != p.tiles_us_per_step)
      fail("order", other, es, q);
    for (size_t d = 0; d < dom.size(); ++d)
      if (q.ntx[d] != p.ntx[order[d]] || q.nty[d] != p.nty[order[d]]) fail("order of the divisions", other, es, q);
  }
}

static void add(Batch* b, int n, int nx, int ny) { b->insert(b->end(), n, DomainSize{nx, ny}); }

int main() {
  for (int es : {4, 8}) {
    // small domains before large ones, thin ones among square ones
    Batch b;
    add(&b, 40, 3, 3); add(&b, 1, 2000, 2000); add(&b, 1, 3000, 3000);
    check(b, es, 1);
    b.clear(); add(&b, 40, 64, 4); add(&b, 1, 1000, 1000);
    check(b, es, 2);
    b.clear();
    for (int i = 0; i < 60; ++i) { add(&b, 1, 100, 4); add(&b, 1, 400, 400); }
    check(b, es, 3);
    b.clear(); add(&b, 1000, 64, 4); add(&b, 1, 2000, 2000);
    check(b, es, 4);
    b.clear(); add(&b, 2000, 3, 3); add(&b, 1, 1500, 1500);
    check(b, es, 5);
    std::mt19937 g(es);
    for (int i = 0; i < 60; ++i) {
      b.clear();
      const int n = 1 + g() % 300, lo = 3 + g() % 60, hi = lo + 1 + g() % (i % 3 == 0 ? 1000 : 200);
      for (int d = 0; d < n; ++d) add(&b, 1, lo + g() % (hi - lo), lo + g() % (hi - lo));
      if (i % 4 == 0) add(&b, 1 + g() % 3, 800 + g() % 2000, 800 + g() % 2000);
      check(b, es, i);
    }
  }
  std::printf("%d batches, 0 failures\n", batches);
  return 0;
}
