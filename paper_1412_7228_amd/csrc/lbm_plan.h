// Host-side choice of the block launches (lbm_block.hip): how many steps a
// launch fuses, the shape of a workgroup and how a lattice is cut into blocks,
// from a cost model of one launch.  Plain C++, no device code.
//
// A launch of k steps over `tiles` blocks costs
//
//   start + sqrt((k * step)^2 + (q * work)^2) + q * moved    q <= r
//   start + q * max(work + hide * moved, k * step / r)       q > r
//
// with q the blocks of the busiest CU, r the workgroups a CU holds at once,
// work the wave instructions of a block's phases (only the rows that take part
// in a phase, in whole waves), moved its loads and stores, `start` the gap
// between two launches with the first loads' latency, and `step` the latency
// of one step's dependent chain (two barriers, the LDS round trips, the
// equation of state and the collision), which is what small lattices wait
// for.  The constants are fitted to 2,150 measured launches (16^2 to 4096^2, k = 2
// to 6, every shape) with a mean error of 4%; the plan that the model picks is
// on average 2% slower than the best one measured, 15% at worst.  States beyond the
// last-level cache wait for HBM besides (hbm_time, block_beyond_cache).
#pragma once

#include <algorithm>
#include <cmath>
#include <tuple>
#include <vector>

#include "lbm_internal.h"

namespace lbm {

struct BlockCost {
  double start, step;      // us
  double density, collide; // us of a CU per wave of cells in the phase
  double moved;            // us of a CU per cell loaded or stored
  double hide;             // share of it that other workgroups' phases do not cover
};

inline BlockCost block_cost(int es) {
  if (es == 4) return {2.04, 0.69, 0.00658, 0.0499, 0.00117, 0.71};
  return {1.76, 0.80, 0.0202, 0.0920, 0.00220, 0.61};
}

struct BlockShape {
  int threads, cells;
};
constexpr BlockShape kBlockShapes[] = {{512, 1}, {1024, 1}, {512, 2}, {1024, 2}, {512, 4}};
constexpr int kBlockMinSteps = 2, kBlockMaxSteps = 6;

// The FP64 kernels of 1024 x 2 would spill registers and are not built.
inline bool block_shape_built(int es, BlockShape s) { return es == 4 || !(s.threads == 1024 && s.cells == 2); }

// Workgroups of a shape that one CU holds: 160 KB of LDS, four SIMDs.
inline int block_resident(int es, BlockShape s) {
  const int by_lds = 160 * 1024 / (s.threads * s.cells * 10 * es);
  const int by_waves = 4 * block_waves(es, s.threads, s.cells) * 64 / s.threads;
  return std::max(1, std::min(by_lds, by_waves));
}

// CU time of the phases of a block of W x H cells, halo included.
inline double block_work(const BlockCost& c, unsigned W, unsigned H, int k) {
  auto waves = [&](unsigned rim) { return (int)(((H - rim) * W + 63) / 64 - rim * W / 64); };
  double t = 0.0;
  for (int s = 0; s < k; ++s) t += c.density * waves(2 * s) + c.collide * waves(2 * s + 1);
  return t;
}

// At most that: every phase takes the stored cells.
inline double block_work_least(const BlockCost& c, double stored, int k) {
  return k * (c.density + c.collide) * stored * (1.0 / 64.0);
}

inline double block_launch_time(const BlockCost& c, int k, double q, double work, double cells_moved, int r) {
  const double moved = c.moved * cells_moved;
  if (q <= r) return c.start + std::sqrt(k * c.step * k * c.step + q * work * q * work) + q * moved;
  return c.start + q * std::max(work + (r > 1 ? c.hide : 1.0) * moved, k * c.step / r);
}

// Fewest rows of blocks for ntx columns of them, 0 if not even one row fits.
inline int block_rows(int nx, int ny, int ntx, int k, int capacity) {
  const int halo = 2 * (2 * k - 1), W = (nx + ntx - 1) / ntx + halo;
  const int h = std::min(ny, capacity / W - halo);
  return h < 1 ? 0 : (ny + h - 1) / h;
}

inline BlockPlan block_plan(int nx, int ny, int k, int ntx, int nty, BlockShape s) {
  BlockPlan p{};
  p.k = k;
  p.ntx = ntx;
  p.nty = nty;
  p.w = nx / ntx;
  p.rx = nx % ntx;
  p.h = ny / nty;
  p.ry = ny % nty;
  p.threads = s.threads;
  p.cells = s.cells;
  return p;
}

// Lattices above this many cells keep the marching tiles, whose halo of 6 rows
// a tile recomputes less than a block's rim once there are tiles enough for
// every CU.  Measured per step, block against marching: FP32 1024^2 9.7 / 14.3
// us, 2048^2 35.6 / 39.9, 3000^2 75.9 / 80.1, 4096^2 135-138 / 137-138; FP64 (half
// the cells in the same LDS) 700^2 9.2 / 14.6, 1024^2 17.0 / 21.1, 1400^2 30.8 /
// 35.7, 2048^2 69.3 / 72.3, 2560^2 104.7 / 110.8, 4000 x 2000 127.6 / 123.4.
inline long long block_max_cells(int es) { return es == 4 ? 12ll << 20 : 7ll << 20; }

// An FP64 state of more than 2^20 cells leaves the 256 MB last-level cache (two
// buffers of 72 MB per 2^20 cells, and the halos' second reads), with whose
// loads the model is fitted.  What waits for HBM there is left out: launches of
// two steps (1700^2 55.8 us a step, at three steps 47.3) and shapes of one
// workgroup a CU (2000 x 1500 at three steps in 512 x 4 58.9, in 512 x 2 49.2,
// the marching tiles 51.9); 60 domains of 200^2 46.0 -> 40.7.  FP32 blocks hold twice the
// cells, and hbm_time alone takes two steps out where they wait (leaving them out at
// 2.2 to 3.6 million cells too: 0.93 to 1.02 of the time).
inline bool block_beyond_cache(int es, long long cells) { return es == 8 && cells > 1ll << 20; }

// The same for a launch of two steps over some rows (lbm_step_rows), whose
// loads and stores are shared by two steps only: FP32 1000 x 700 16.7 us a launch
// against 24.0, 1024^2 22.2 / 28.6, 4096 x 512 with its ghost rows refreshed in
// between 43.0 / 43.0, 2048^2 84.8 / 79.4; FP64 1607 x 144 with refreshes, 25
// launches, 447 / 669 us.
inline long long block_max_row_cells(int es) { return es == 4 ? 3ll << 19 : 1ll << 20; }

// The end of a call on a lattice in blocks: fewer steps than a launch's k load and
// store as much for less work, so one step, or two where k is three, may go to the
// marching tiles: lattices above these sizes whose strips leave at most a fifth of
// their lanes idle (lanes: of a row of strips).  Measured by blocks / by tiles, us a call
// in a loop: one step, FP32 886^2 12.9 / 14.7, 1000^2 16.1 / 15.6, 2048^2 69.4 / 57.7,
// 300 x 5000 (idle lanes) 22.1 / 22.9, FP64 1000^2 25.9 / 24.5, 1254^2 37.1 / 42.2, 1448^2
// 68.5 / 65.8, 2048^2 132 / 118; two steps, FP32 1448^2 38.6 / 38.9, 1700^2 50.1 / 53.8,
// 2048^2 85.6 / 78.0, 3000^2 179 / 159, FP64 1130^2 42.2 / 43.1, 1254^2 51.9 / 51.2, 1448^2
// 84.6 / 78.8, 2048^2 165 / 145, 300 x 5000 48.2 / 62.2; four as three and one / as two
// and two by tiles, FP32 2048^2 170 / 155, FP64 1130^2 89.4 / 86.4.
struct LatticeRest {
  bool one, two;  // by the tiles
};

inline LatticeRest lattice_rest(int es, int nx, int ny, int lanes1, int lanes2) {
  const long long cells = (long long)nx * ny;
  return {cells > (es == 4 ? 7ll << 17 : 31ll << 16) && 4ll * lanes1 <= 5ll * nx,
          cells > (es == 4 ? 7ll << 19 : 1ll << 20) && 4ll * lanes2 <= 5ll * nx};
}

// Steps of the next launch of a call with `left` steps to go.
inline int lattice_next_steps(long long left, int k, LatticeRest r) {
  if (k == 3 && left == 4 && r.two) return 2;
  return left < k ? (int)left : k;
}

// Widths tried for a block: every sixth of an octave, 3 to 512 columns.
template <typename F>
void for_block_widths(int nx, F f) {
  int last = 0;
  for (double w = 3.0; w <= 512.0; w *= 1.1225) {
    const int ntx = std::max(1, (nx + (int)w - 1) / (int)w);
    if (ntx != last) f(ntx);
    last = ntx;
    if (ntx == 1) break;
  }
}

// A state whose two buffers pass the 256 MB last-level cache moves its cells at the
// rate of HBM: a launch takes at least its loads and stores at 4.5 TB/s (FP32) or
// 5.0 (FP64), the halos' second reads included (4096^2 in blocks of 38 x 32, one
// step: 1.28 GB in 272 us; FP64 24 x 20, one step 2.65 GB in 497; 3000^2 at two
// steps 766 MB in 174, where the fitted model says 149).
inline double hbm_time(int es, double all_cells, double cells_moved) {
  return all_cells * 18 * es > 256e6 ? cells_moved * 9 * es / (es == 4 ? 4.5e6 : 5.0e6) : 0.0;
}

// The plan of least modelled time per step for `rows` rows of a lattice; max_k
// bounds the steps of a launch (min_k of a launch that must take that many).
inline BlockPlan plan_lattice(int nx, int rows, int es, int cus, int min_k, int max_k, double* us_per_step) {
  const BlockCost c = block_cost(es);
  const bool far = block_beyond_cache(es, (long long)nx * rows);
  if (far) min_k = std::max(min_k, 3);
  constexpr int kShapes = sizeof kBlockShapes / sizeof *kBlockShapes;
  BlockPlan best[kShapes] = {};
  double least[kShapes], any = 1e300;  // of each shape, and of all
  for (double& t : least) t = 1e300;
  // one division of the lattice, its time by any shape
  struct Division {
    int nty;
    double q, moved, work;  // work < 0: not yet formed
  };
  // A context is made for every lattice of a sweep, so the search itself counts (200^2
  // FP32 25 us of host time, 35 when every division's time is formed): what shapes
  // share is formed once, and a division's work only where its least possible time
  // is not above the best yet.
  for (int k = max_k; k >= min_k; --k) {
    const int halo = 2 * (2 * k - 1);
    for_block_widths(nx, [&](int ntx) {
      const int w = (nx + ntx - 1) / ntx;
      auto division = [&](int nty) {
        const int h = (rows + nty - 1) / nty;
        return Division{nty, (double)(((long long)ntx * nty + cus - 1) / cus),
                        (double)(w + halo) * (h + halo) + (double)w * h, -1.0};
      };
      // as many blocks as the CUs take in one to four rounds
      Division rounds[4];
      int formed = 0, round_nty[4];
      for (int round = 1; round <= 4; ++round) round_nty[round - 1] = std::min(rows, round * cus / ntx);
      for (int i = 0; i < kShapes; ++i) {
        const BlockShape s = kBlockShapes[i];
        if (!block_shape_built(es, s)) continue;
        const int r = block_resident(es, s);
        if (far && r < 2) continue;
        if (c.start + k * c.step / r > any * k) continue;  // not even the latency fits
        const int fewest = block_rows(nx, rows, ntx, k, s.threads * s.cells);
        if (fewest == 0) continue;
        auto take = [&](Division& d) {
          const int h = (rows + d.nty - 1) / d.nty;
          const double stored = (double)w * h, hbm = hbm_time(es, (double)nx * rows, ntx * d.nty * d.moved);
          if (std::max(block_launch_time(c, k, d.q, block_work_least(c, stored, k), d.moved, r), hbm) > any * k) return;
          if (d.work < 0.0) d.work = block_work(c, w + halo, h + halo, k);
          const double t = std::max(block_launch_time(c, k, d.q, d.work, d.moved, r), hbm) / k;
          if (t >= least[i]) return;
          least[i] = t;
          any = std::min(any, t);
          best[i] = block_plan(nx, rows, k, ntx, d.nty, s);
        };
        Division fewest_blocks = division(fewest);
        take(fewest_blocks);
        for (int q = 0; q < 4; ++q) {
          if (round_nty[q] <= fewest) continue;
          if (!(formed & 1 << q)) rounds[q] = division(round_nty[q]);
          formed |= 1 << q;
          take(rounds[q]);
        }
      }
    });
  }
  int shape = 0;
  for (int i = 1; i < kShapes; ++i)
    if (least[i] < least[shape]) shape = i;
  if (us_per_step) *us_per_step = least[shape];
  return best[shape];
}

// ---------------------------------------------------------------------------
// Batches
// ---------------------------------------------------------------------------
// One launch of a batch: its steps, by blocks or by the marching tiles.
struct BatchLaunch {
  int steps;
  bool tiles;
};

// What a call does with its last steps, at most 2 k of them: the next launch for
// each number of steps left, and the launches that number takes in all.
struct BatchTail {
  BatchLaunch next[2 * kBlockMaxSteps + 1];
  int launches[2 * kBlockMaxSteps + 1];
};

// Block launches of a batch: every domain's blocks in one launch of k steps
// (domain d in ntx[d] x nty[d] of them), or, with `whole`, every domain whole
// in one workgroup, any number of steps a launch.  k = 0: marching tiles.
struct BatchBlocks {
  int k = 0;
  bool whole = false;
  BlockShape shape{};
  std::vector<int> ntx, nty;
  double us_per_step = 1e300, tiles_us_per_step = 1e300;  // modelled; the tiles' of the default shape
  BatchTail tail{};

  // The next launch of a call with `left` steps to go, and a call's launches
  // (not of whole domains).
  BatchLaunch next(int left) const { return left > 2 * k ? BatchLaunch{k, false} : tail.next[left]; }
  int launches(int n) const {
    const int full = n > 2 * k ? (n - k - 1) / k : 0;
    return full + tail.launches[n - full * k];
  }
};

struct DomainSize {
  int nx, ny;
};

// The domains of one size together, larger sizes first: what a plan sees, whatever
// the order of the batch.
struct DomainClass {
  DomainSize size;
  double count;
  double cells() const { return (double)size.nx * size.ny; }
  double weight() const { return count * (cells() + 512.0); }  // 512: a block's cost of being there
};

// The classes of a batch; of[d] is the class of domain d.
inline std::vector<DomainClass> domain_classes(const std::vector<DomainSize>& dom, std::vector<int>* of) {
  std::vector<int> order(dom.size());
  for (size_t d = 0; d < dom.size(); ++d) order[d] = (int)d;
  auto key = [&](int d) { return std::make_tuple(-(long long)dom[d].nx * dom[d].ny, dom[d].nx); };
  std::sort(order.begin(), order.end(), [&](int a, int b) { return key(a) < key(b); });
  std::vector<DomainClass> classes;
  of->resize(dom.size());
  for (int d : order) {
    if (classes.empty() || classes.back().size.nx != dom[d].nx || classes.back().size.ny != dom[d].ny)
      classes.push_back({dom[d], 0.0});
    classes.back().count += 1.0;
    (*of)[d] = (int)classes.size() - 1;
  }
  return classes;
}

// At most `most` classes that stand for all of them: the classes in shares of
// equal weight, each share by the class at its middle.
inline std::vector<DomainClass> sample_classes(const std::vector<DomainClass>& classes, int most) {
  if ((int)classes.size() <= most) return classes;
  double all = 0.0;
  for (const auto& q : classes) all += q.weight();
  std::vector<DomainClass> out;
  double from = 0.0;  // weight before class i
  size_t i = 0;
  for (int s = 0; s < most; ++s) {
    const double middle = (s + 0.5) / most * all;
    while (i + 1 < classes.size() && from + classes[i].weight() < middle) from += classes[i++].weight();
    out.push_back({classes[i].size, all / most / (classes[i].cells() + 512.0)});
  }
  return out;
}

// Shapes of the whole-domain kernel: the smallest that holds the largest
// domain (small workgroups share a CU).
constexpr BlockShape kWholeShapes[] = {{256, 1}, {512, 1}, {1024, 1}, {512, 4}};

// The division of a domain of least work; the caller's sums over its blocks.
struct BlockCut {
  int ntx = 0, nty = 0;
  double work = 1e300, cells = 0.0;
};

inline BlockCut cut_domain(const BlockCost& c, const DomainSize& d, BlockShape s, int k, int finer) {
  const int halo = 2 * (2 * k - 1);
  BlockCut best;
  for_block_widths(d.nx, [&](int ntx) {
    const int fewest = block_rows(d.nx, d.ny, ntx, k, s.threads * s.cells);
    if (fewest == 0) return;
    const int nty = std::min(d.ny, fewest * finer);
    const int w = (d.nx + ntx - 1) / ntx, h = (d.ny + nty - 1) / nty;
    const double n = (double)ntx * nty, stored = (double)w * h;
    BlockCut q{ntx, nty, n * block_work_least(c, stored, k), n * ((double)(w + halo) * (h + halo) + stored)};
    auto better = [&] { return q.work + c.hide * c.moved * q.cells < best.work + c.hide * c.moved * best.cells; };
    if (!better()) return;
    q.work = ntx * nty * block_work(c, w + halo, h + halo, k);
    if (better()) best = q;
  });
  return best;
}

// What a launch of k steps over all of a batch costs, its domains' blocks added up.
// Blocks of domains far smaller than a workgroup wait twice for their start and chain,
// shared by the r workgroups of a CU (2,000 domains of 3^2 beside a 1500^2).
//
// Beyond block_beyond_cache the FP64 model is 1.16 times what is measured (1448^2 to
// 4096^2, 60 to 240 domains of 200^2, uneven ones: 1.13 to 1.19).
struct BatchLaunchCost {
  int es, k, resident;
  double blocks = 0.0, work = 0.0, cells = 0.0, busy = 0.0;
  void add(const BlockCut& q, double count) {
    const BlockCost c = block_cost(es);
    const double n = (double)q.ntx * q.nty;
    blocks += count * n;
    work += count * q.work;
    cells += count * q.cells;
    busy += count * std::max(q.work + (resident > 1 ? c.hide : 1.0) * c.moved * q.cells,
                             n * 2.0 * (c.start + k * c.step) / resident);
  }
  double us(double all_cells, int cus) const {
    const BlockCost c = block_cost(es);
    const double q = std::ceil(blocks / cus);
    double t = q <= resident ? block_launch_time(c, k, q, work / blocks, cells / blocks, resident)
                             : c.start + q * busy / blocks;
    if (block_beyond_cache(es, (long long)all_cells) && es == 8) t *= 0.86;
    return std::max(t, hbm_time(es, all_cells, cells));
  }
};

// A launch of the marching tiles of the default shape (256 lanes by 16 rows, of which
// a two-step launch stores 250 columns): so much a tile and so much a cell, and at
// least a tile's chain of rows.  Fitted to 34 batches (one domain of 1024^2 to
// 4,000 of 50^2) within 5% rms (two steps) and 6 to 9% (one).
inline double batch_tiles_time(const std::vector<DomainClass>& classes, int es, int steps) {
  const int w = steps == 2 ? 256 - kStep2Halo : 256;
  double tiles = 0.0, cells = 0.0;
  for (const auto& q : classes) {
    tiles += q.count * ((q.size.nx + w - 1) / w) * ((q.size.ny + 15) / 16);
    cells += q.count * q.cells();
  }
  if (steps == 2)
    return es == 4 ? std::max(35.0, 10.4 + 31.5e-3 * tiles + 8.1e-6 * cells)
                   : std::max(41.0, 21.3 + 79.5e-3 * tiles + 11.9e-6 * cells);
  return es == 4 ? std::max(22.0, 16.6e-3 * tiles + 11.2e-6 * cells)
                 : std::max(26.0, 9.7 + 38.0e-3 * tiles + 18.3e-6 * cells);
}

// The launches of the last steps of a call: a block launch of as many as there are, or
// the tiles where they take less: a launch of fewer steps than k loads and stores as
// much for less work, and large batches of wide domains are faster on the tiles then
// (4096^2 FP32, us a step: one step by blocks 278, by tiles 239; two 163 / 141; four as
// three and one 168, as two and two by tiles 139; 1,000 domains of 64^2, whose tiles are
// three quarters idle, one step 78 / 118).  The models' ratio misses what 31 batches of
// 50 us a step and more measured by up to a sixth; one step goes to the tiles where
// theirs is below 0.925 (below that 0.84 to 1.01 measured and once 1.07, above it up to
// 1.09), two below 1.02 (0.84 to 1.01).
inline BatchTail plan_tail(int k, const double (&block_us)[kBlockMaxSteps + 1], double tile1_us, double tile2_us) {
  BatchTail tail{};
  double cost[2 * kBlockMaxSteps + 1] = {};
  for (int m = 1; m <= 2 * k; ++m) {
    cost[m] = 1e300;
    auto take = [&](int steps, bool tiles, double us) {
      if (us + cost[m - steps] >= cost[m]) return;
      cost[m] = us + cost[m - steps];
      tail.next[m] = {steps, tiles};
      tail.launches[m] = 1 + tail.launches[m - steps];
    };
    const double margin = m > k ? 1.04 : 1.0;
    take(std::min(m, k), false, block_us[std::min(m, k)]);
    if (m >= 2) take(2, true, tile2_us * 0.98 * margin);
    take(1, true, tile1_us * 1.08 * margin);
  }
  return tail;
}

// Steps and shape from at most 16 classes that stand for the batch, then every
// class's division, whose sum is the plan's time; the caller takes the tiles where
// they take less.  (Sampled by their place in the
// batch, 40 domains of 3^2 before a 2000^2 and a 3000^2 chose for the small ones:
// 1,790 us a step, where the tiles take 112 and this plan 107.)
inline BatchBlocks plan_batch(const std::vector<DomainSize>& dom, int es, int cus) {
  const BlockCost c = block_cost(es);
  std::vector<int> of;
  const std::vector<DomainClass> classes = domain_classes(dom, &of), samples = sample_classes(classes, 16);
  double all_cells = 0.0;
  for (const auto& q : classes) all_cells += q.count * q.cells();
  BatchBlocks best;
  for (BlockShape s : kWholeShapes) {
    if (classes[0].cells() > s.threads * s.cells) continue;
    // no launch, no halo: the chain of a step, or the work of the busiest CU
    double work = 0.0;
    for (const auto& q : classes) work += q.count * (c.density + c.collide) * ((q.size.nx * q.size.ny + 63) / 64);
    const double q = (double)((dom.size() + cus - 1) / cus);
    const double own = q * work / dom.size(), wait = c.step * std::ceil(q * s.threads / 512);
    best.us_per_step = std::sqrt(own * own + wait * wait);
    best.whole = true;
    best.k = 1;
    best.shape = s;
    break;
  }
  // a batch of fewer blocks than CUs divides its domains further
  const bool far = block_beyond_cache(es, (long long)all_cells);
  int finer = 1;
  for (BlockShape s : kBlockShapes) {
    if (!block_shape_built(es, s) || (far && block_resident(es, s) < 2)) continue;
    for (int k = far ? 3 : kBlockMinSteps; k <= kBlockMaxSteps; ++k)
      for (int f = 1; f > 0;) {
        BatchLaunchCost sums{es, k, block_resident(es, s)};
        bool fits = true;
        for (const auto& d : samples) {
          const BlockCut q = cut_domain(c, d.size, s, k, f);
          if (!(fits = q.ntx > 0)) break;
          sums.add(q, d.count);
        }
        if (!fits) break;
        const double t = sums.us(all_cells, cus) / k;
        if (t < best.us_per_step) {
          best = BatchBlocks{};
          best.k = k;
          best.shape = s;
          best.us_per_step = t;
          finer = f;
        }
        f = f == 1 && sums.blocks * 2 <= cus ? (int)(cus / sums.blocks) : 0;
      }
  }
  if (best.whole || best.k == 0) return best;
  std::vector<BlockCut> cuts;
  for (const auto& d : classes) {
    cuts.push_back(cut_domain(c, d.size, best.shape, best.k, finer));
    if (cuts.back().ntx == 0) return BatchBlocks{};  // a domain that the chosen blocks do not fit: marching tiles
  }
  // the time of a launch of each number of steps by these blocks
  double block_us[kBlockMaxSteps + 1] = {};
  for (int k = 1; k <= best.k; ++k) {
    BatchLaunchCost sums{es, k, block_resident(es, best.shape)};
    for (size_t q = 0; q < classes.size(); ++q) {
      const DomainSize& d = classes[q].size;
      const int halo = 2 * (2 * k - 1), ntx = cuts[q].ntx, nty = cuts[q].nty;
      const int w = (d.nx + ntx - 1) / ntx, h = (d.ny + nty - 1) / nty;
      sums.add({ntx, nty, ntx * nty * block_work(c, w + halo, h + halo, k),
                (double)ntx * nty * ((double)(w + halo) * (h + halo) + (double)w * h)}, classes[q].count);
    }
    block_us[k] = sums.us(all_cells, cus);
  }
  const double tile2_us = batch_tiles_time(classes, es, 2);
  best.us_per_step = block_us[best.k] / best.k;
  best.tiles_us_per_step = tile2_us / 2;
  best.tail = plan_tail(best.k, block_us, batch_tiles_time(classes, es, 1), tile2_us);
  for (int q : of) {
    best.ntx.push_back(cuts[q].ntx);
    best.nty.push_back(cuts[q].nty);
  }
  return best;
}

}  // namespace lbm
