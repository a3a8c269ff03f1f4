// FP64 read-out of a state: density/psi fields, velocity, distribution planes,
// and the deterministic reduction of the observables (mass, momentum,
// extremes, faults) used by the Laplace-law measurement (Eq. 22).
// Off the hot path: these run only when the caller asks for observables or fields.
#include <mutex>

#include "lbm_tile.h"

namespace lbm {

constexpr int kRedThreads = 256;

// rho = sum_a f_a(x) of the current (streamed) state, U and psi in FP64.
template <typename T, int EOS>
__global__ void k_density_fields(const T* __restrict__ f, const Geometry geo, const DevC<double> c,
                                 double* __restrict__ work) {
  const long long n = (long long)geo.nx * geo.ny;
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int y = (int)(i / geo.nx), x = (int)(i - (long long)y * geo.nx);
  double r = 0.0;
#pragma unroll
  for (int a = 0; a < 9; ++a) r += (double)f[state_index(geo, a, x, y)];
  const double U = eos_U<EOS>(r, c);
  work[i] = r;
  work[n + i] = U;
  work[2 * n + i] = psi_of(U, c);
}

// rho alone, into out[ny][nx] (device or pinned host memory).
template <typename T>
__global__ void k_density(const T* __restrict__ f, const Geometry geo, double* __restrict__ out) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (long long)geo.nx * geo.ny) return;
  const int y = (int)(i / geo.nx), x = (int)(i - (long long)y * geo.nx);
  double r = 0.0;
#pragma unroll
  for (int a = 0; a < 9; ++a) r += (double)f[state_index(geo, a, x, y)];
  out[i] = r;
}

// Force of Eq. (9) at a cell from U and psi at the cell (index 0) and at its
// eight neighbours x + e_a (index a) (the weights 1/3, 1/12 applied as
// 12 sum_a w_a phi e_a), and the momentum j of the cell's distributions g.
__device__ inline void force_core(const double (&Un)[9], const double (&Pn)[9], const DevC<double>& c, double& Fx,
                                  double& Fy) {
  const double gUx = 4.0 * (Un[1] - Un[3]) + ((Un[5] - Un[7]) + (Un[8] - Un[6]));
  const double gUy = 4.0 * (Un[2] - Un[4]) + ((Un[5] - Un[7]) + (Un[6] - Un[8]));
  const double gPx = 4.0 * (Pn[1] - Pn[3]) + ((Pn[5] - Pn[7]) + (Pn[8] - Pn[6]));
  const double gPy = 4.0 * (Pn[2] - Pn[4]) + ((Pn[5] - Pn[7]) + (Pn[6] - Pn[8]));
  const double fpp = c.fP * Pn[0];
  Fx = c.fU * gUx + fpp * gPx;
  Fy = c.fU * gUy + fpp * gPy;
}

__device__ inline void momentum_core(const double (&g)[9], double& jx, double& jy) {
  jx = (g[1] - g[3]) + ((g[5] - g[7]) + (g[8] - g[6]));
  jy = (g[2] - g[4]) + ((g[5] - g[7]) + (g[6] - g[8]));
}

// Offsets e_a of the lattice velocities, in the order of the distributions.
__device__ __forceinline__ int ex_of(int a) { return (a == 1 || a == 5 || a == 8) ? 1 : ((a == 3 || a == 6 || a == 7) ? -1 : 0); }
__device__ __forceinline__ int ey_of(int a) { return (a == 2 || a == 5 || a == 6) ? 1 : ((a == 4 || a == 7 || a == 8) ? -1 : 0); }

// rho = sum_a f_a(x, y) of the current (streamed) state in FP64, summed in
// plane order (the order every read-out uses).
template <typename T>
__device__ inline double cell_density(const T* __restrict__ f, const Geometry& geo, int x, int y) {
  double r = 0.0;
#pragma unroll
  for (int a = 0; a < 9; ++a) r += (double)f[state_index(geo, a, x, y)];
  return r;
}

template <typename T>
__device__ inline void cell_distributions(const T* __restrict__ f, const Geometry& geo, int x, int y,
                                          double (&g)[9]) {
#pragma unroll
  for (int a = 0; a < 9; ++a) g[a] = (double)f[state_index(geo, a, x, y)];
}

// Force and momentum at (x, y) from the FP64 U/psi fields of k_density_fields.
template <typename T>
__device__ inline void force_and_momentum(const T* __restrict__ f, const Geometry& geo,
                                          const DevC<double>& c, const double* __restrict__ work,
                                          int x, int y, double& Fx, double& Fy, double& jx,
                                          double& jy) {
  const long long n = (long long)geo.nx * geo.ny;
  const double* U = work + n;
  const double* psi = work + 2 * n;
  double Un[9], Pn[9], g[9];
#pragma unroll
  for (int a = 0; a < 9; ++a) {
    const long long i = (long long)wrap_(y + ey_of(a), geo.ny) * geo.nx + wrap_(x + ex_of(a), geo.nx);
    Un[a] = U[i];
    Pn[a] = psi[i];
  }
  cell_distributions(f, geo, x, y, g);
  force_core(Un, Pn, c, Fx, Fy);
  momentum_core(g, jx, jy);
}

template <typename T>
__global__ void k_velocity(const T* __restrict__ f, const Geometry geo, const DevC<double> c,
                           const double* __restrict__ work, int comp, double* __restrict__ out) {
  const long long n = (long long)geo.nx * geo.ny;
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int y = (int)(i / geo.nx), x = (int)(i - (long long)y * geo.nx);
  double Fx, Fy, jx, jy;
  force_and_momentum(f, geo, c, work, x, y, Fx, Fy, jx, jy);
  out[i] = (comp == 0 ? jx + 0.5 * Fx : jy + 0.5 * Fy) / work[i];
}

// A lane's share of the observables, and the largest |v|^2 its wave has seen.
struct ObsSum {
  double mass, mx, my, lo, hi, v2, wave_v2;
  unsigned n_domain, n_bad;
};

// One cell's contribution: mass, momentum (j + F/2), density extremes, max
// |v|^2, and the fault counts.  The two FP64 divisions of v = (j + F/2) / rho
// are a quarter of the arithmetic, and a cell can only raise the maximum if
// (j + F/2)^2 > max rho^2 (up to rounding: the bound is lowered by 1e-12), so a
// wave divides only where one of its lanes passes that test against the
// wave's maximum, on 4 rows of 35 or so.  Squares that are not normal numbers
// (densities beyond 1e+-154, momenta below 1e-154) decide nothing: such cells
// divide, but for those whose momentum is zero.
__device__ __forceinline__ void accumulate_cell(ObsSum& s, bool own, double r, double U, double Fx, double Fy,
                                                double jx, double jy) {
  const double mx = jx + 0.5 * Fx, my = jy + 0.5 * Fy;
  if (own) {
    s.mass += r;
    s.mx += mx;
    s.my += my;
    s.lo = fmin(s.lo, r);
    s.hi = fmax(s.hi, r);
    s.n_domain += U <= 0.0 ? 0u : 1u;               // U > 0 (or NaN)
    s.n_bad += r > 0.0 && isfinite(r) ? 0u : 1u;    // rho <= 0 or not finite
  }
  const double m2 = mx * mx + my * my, r2 = r * r;
  constexpr int kNormal = 0x100 | 0x008;  // v_cmp_class: positive, negative normal
  const bool m_normal = __builtin_amdgcn_class(m2, kNormal), r_normal = __builtin_amdgcn_class(r2, kNormal);
  const bool above = m2 > s.wave_v2 * r2 * (1.0 - 1e-12) || !r_normal;
  if (__any(own && (above || !m_normal)) &&
      __any(own && (above || (!m_normal && (mx != 0.0 || my != 0.0))))) {
    const double vx = mx / r, vy = my / r;
    const double v2 = vx * vx + vy * vy;
    if (own && v2 == v2) s.v2 = fmax(s.v2, v2);
    double w = s.v2;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) w = fmax(w, __shfl_xor(w, o));
    s.wave_v2 = w;
  }
}

// Tree reduction of the block's accumulators in a fixed order; thread q <
// kNumRed writes entry q of the block's result to out[q].
__device__ inline void block_reduce_store(const double (&acc)[kNumRed], double (&sh)[kNumRed][kRedThreads],
                                          double* __restrict__ out) {
#pragma unroll
  for (int q = 0; q < kNumRed; ++q) sh[q][threadIdx.x] = acc[q];
  __syncthreads();
  for (int stride = kRedThreads / 2; stride > 0; stride >>= 1) {
    if ((int)threadIdx.x < stride) {
      const int o = threadIdx.x + stride;
      sh[0][threadIdx.x] += sh[0][o];
      sh[1][threadIdx.x] += sh[1][o];
      sh[2][threadIdx.x] += sh[2][o];
      sh[3][threadIdx.x] = fmin(sh[3][threadIdx.x], sh[3][o]);
      sh[4][threadIdx.x] = fmax(sh[4][threadIdx.x], sh[4][o]);
      sh[5][threadIdx.x] = fmax(sh[5][threadIdx.x], sh[5][o]);
      sh[6][threadIdx.x] += sh[6][o];
      sh[7][threadIdx.x] += sh[7][o];
    }
    __syncthreads();
  }
  if (threadIdx.x < kNumRed) out[threadIdx.x] = sh[threadIdx.x][0];
}

// ---------------------------------------------------------------------------
// Observables: one pass over the distributions.  A workgroup marches down a
// tile of 254 columns (256 lanes with the two neighbour columns) and H rows:
// it gathers a row's populations, forms rho, U and psi into a ring of four LDS
// rows, and after one barrier the row before has its 3 x 3 stencil and adds to
// the lanes' accumulators.  Nothing but the partial sums goes to HBM, and f is
// read (H + 2) / H times.
//
// Bound by HBM on large lattices: 4096^2 FP32 reads 0.65 GB in 126 us (5.1 TB/s;
// FP64 1.3 GB in 210 us) in place of the 2.1 GB in 450 us that rho, U and psi as
// FP64 fields in HBM took (written, read back as stencils, f read twice).  Small
// ones wait for a tile's chain of rows, hence tiles of 4 rows while that leaves
// CUs idle.  A batch's domains go in one launch (256 slabs of 64 x 4: 8.6 ms of
// launches, copies and waits one by one, 0.03 ms together).  The partial sums
// are added in a fixed order (rows of a tile, tiles of a block, blocks).
// ---------------------------------------------------------------------------
constexpr int kObsWidth = kRedThreads - 2;
constexpr int kObsMaxBlocks = 4096;  // blocks beyond take several tiles each

// Lattices of up to this many columns leave half of a tile's lanes idle and more: there
// a workgroup takes two tiles and more, one above the other, side by side in its lanes
// (obs_tile_narrow).  A call with one tile and so: 3 x 140001 FP32 190 and 53 us, 32 x
// 32768 69 / 35, 64 x 16384 50 / 37, 100 x 20000 56 / 49, 1,000 domains of 64^2 205 / 124.
constexpr int kObsNarrow = kRedThreads / 2 - 2;

struct ObsTiles {
  int strips, rows, tiles;  // columns of tiles, rows of a tile, tiles (groups of them) in all
  int groups;               // tiles side by side in a workgroup's lanes (1: wide lattices)
};

// Rows that give at most 2,048 tiles, two rounds of the four workgroups a CU
// holds (a third, nearly empty round costs a third of the time: 4096^2 in 32
// rows, 2,176 tiles); at least 4, and at most 40, beyond which a round's end
// weighs less than the registers' reuse gains.
static ObsTiles obs_tiles(const Geometry& g) {
  const int groups = g.nx <= kObsNarrow ? kRedThreads / (g.nx + 2) : 1;
  const int strips = (g.nx + kObsWidth - 1) / kObsWidth;
  const int blocks = (strips < 2048 ? 2048 / strips : 1) * groups;
  const int most = (g.ny + blocks - 1) / blocks, rows = most < 4 ? 4 : (most > 40 ? 40 : most);
  const int high = rows * groups;
  return ObsTiles{strips, rows, strips * ((g.ny + high - 1) / high), groups};
}

template <typename T, int EOS, bool BIG>
__device__ __forceinline__ void obs_tile(const T* __restrict__ f, const Geometry& geo, const DevC<double>& c, int xs,
                                         int y0, int H, ObsSum& sum, double2 (*ring)[kRedThreads]) {
  const int nx = geo.nx, ny = geo.ny, tx = threadIdx.x;
  const int u = xs - 1 + tx, x = (u + nx) % nx;
  const unsigned sz = sizeof(T), ox = x * sz;
  const unsigned oxm = (x == 0 ? nx - 1 : x - 1) * sz, oxp = (x == nx - 1 ? 0 : x + 1) * sz;
  const bool own = tx >= 1 && tx <= kObsWidth && u < nx;
  Planes<BIG> pa;
  pa.init(f, geo.pitch * sz, (unsigned)(geo.row * sz), (unsigned long long)geo.ny * geo.row * sz);
  auto wrap_row = [&](int y) { return y < 0 ? y + ny : (y >= ny ? y - ny : y); };
  struct Row {
    double r, U, jx, jy;
  } now{}, before{};
  const int n = H + 2;
  T P[9], Q[9];
  auto gather_row = [&](int y, T(&g)[9]) {
    gather(pa, wrap_row(y), wrap_row(wrap_row(y) - 1), wrap_row(wrap_row(y) + 1), ox, oxm, oxp, g);
  };
  gather_row(y0 - 1, P);
  gather_row(y0, Q);
  __syncthreads();  // the ring's last readers (the tile before) are done
  // two sets of populations take turns: once a row's density and momentum are
  // formed, its set takes the row after next.  Rows past the last (the two
  // gathered ahead, the one that makes n even) are row y0 + H again and add
  // nothing: with the loads under a condition the compiler copies the sets at
  // the end of the loop, and waits for the loads there
  auto iteration = [&](int i, T(&g)[9]) {
    double d[9];
    now.r = 0.0;
#pragma unroll
    for (int a = 0; a < 9; ++a) {
      d[a] = (double)g[a];
      now.r += d[a];
    }
    momentum_core(d, now.jx, now.jy);
    gather_row(y0 + min(i + 1, H), g);
    now.U = eos_U<EOS>(now.r, c);
    ring[i & 3][tx] = double2{now.U, psi_of(now.U, c)};
    __syncthreads();
    if (i >= 2) {
      const int l = tx == 0 ? 0 : tx - 1, q = tx == kRedThreads - 1 ? tx : tx + 1;  // the rim's lanes add nothing
      const double2 *nr = ring[i & 3], *mr = ring[(i - 1) & 3], *sr = ring[(i - 2) & 3];
      const double2 v[9] = {mr[tx], mr[q], nr[tx], mr[l], sr[tx], nr[q], nr[l], sr[l], sr[q]};
      double Un[9], Pn[9], Fx, Fy;
#pragma unroll
      for (int a = 0; a < 9; ++a) {
        Un[a] = v[a].x;
        Pn[a] = v[a].y;
      }
      force_core(Un, Pn, c, Fx, Fy);
      accumulate_cell(sum, own && i < n, before.r, before.U, Fx, Fy, before.jx, before.jy);
    }
    before = now;
  };
#pragma unroll 1
  for (int i = 0; i < n; i += 2) {
    iteration(i, P);
    iteration(i + 1, Q);
  }
}

// Tiles y0, y0 + H, ... of a narrow lattice side by side, each with the two
// neighbour columns: obs_tile with the rows its lanes' own.  They are gathered one
// after the other at three byte offsets that move on by a row, of 32 bits below 4 GiB:
// nine 64-bit addresses formed afresh for each row took 71.1 us a call on 64 x 65536 in
// FP32 where this takes 64.2 (FP64 85.5 / 83.1), 25.2 on 100 x 100 in FP64 (24.8).
template <typename T, int EOS, typename O>
__device__ __forceinline__ void obs_tile_narrow(const T* __restrict__ f, const Geometry& geo, const DevC<double>& c,
                                                int y0, int H, int groups, ObsSum& sum,
                                                double2 (*ring)[kRedThreads]) {
  const int nx = geo.nx, ny = geo.ny, tx = threadIdx.x, wide = nx + 2;
  const int g = tx / wide, u = tx - g * wide - 1, x = (u + nx) % nx;
  const O ox = (O)(x * sizeof(T)), oxm = (O)((x == 0 ? nx - 1 : x - 1) * sizeof(T)),
          oxp = (O)((x == nx - 1 ? 0 : x + 1) * sizeof(T));
  const int from = g < groups ? min(y0 + g * H, ny) : ny, h = min(H, ny - from);  // this lane's rows
  const bool own = u >= 0 && u < nx;
  const long long pitch = geo.pitch;
  auto wrap_row = [&](int y) { return y < 0 ? y + ny : (y >= ny ? y - ny : y); };
  const O row = (O)(geo.row * sizeof(T)), end = row * (O)ny;
  const int first = wrap_row(from - 1);
  O r = row * (O)first, m = row * (O)wrap_row(first - 1), p = row * (O)wrap_row(first + 1);
  struct Row {
    double r, U, jx, jy;
  } now{}, before{};
  const int n = H + 2;
  T P[9], Q[9];
  auto load = [&](int a, O o) {
    return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(f + a * pitch) + o);
  };
  // row from - 1 + min(i, h + 1), for i = 0, 1, 2, ... in turn
  auto gather_row = [&](int i, T(&q)[9]) {
    q[0] = load(0, r + ox);
    q[1] = load(1, r + oxm);
    q[2] = load(2, m + ox);
    q[3] = load(3, r + oxp);
    q[4] = load(4, p + ox);
    q[5] = load(5, m + oxm);
    q[6] = load(6, m + oxp);
    q[7] = load(7, p + oxp);
    q[8] = load(8, p + oxm);
    if (i <= h) {
      m = r;
      r = p;
      p += row;
      if (p == end) p = 0;
    }
  };
  gather_row(0, P);
  gather_row(1, Q);
  __syncthreads();  // the ring's last readers (the tiles before) are done
  auto iteration = [&](int i, T(&q)[9]) {
    double d[9];
    now.r = 0.0;
#pragma unroll
    for (int a = 0; a < 9; ++a) {
      d[a] = (double)q[a];
      now.r += d[a];
    }
    momentum_core(d, now.jx, now.jy);
    gather_row(i + 2, q);
    now.U = eos_U<EOS>(now.r, c);
    ring[i & 3][tx] = double2{now.U, psi_of(now.U, c)};
    __syncthreads();
    if (i >= 2) {
      const int l = tx == 0 ? 0 : tx - 1, e = tx == kRedThreads - 1 ? tx : tx + 1;  // the rim's lanes add nothing
      const double2 *nr = ring[i & 3], *mr = ring[(i - 1) & 3], *sr = ring[(i - 2) & 3];
      const double2 v[9] = {mr[tx], mr[e], nr[tx], mr[l], sr[tx], nr[e], nr[l], sr[l], sr[e]};
      double Un[9], Pn[9], Fx, Fy;
#pragma unroll
      for (int a = 0; a < 9; ++a) {
        Un[a] = v[a].x;
        Pn[a] = v[a].y;
      }
      force_core(Un, Pn, c, Fx, Fy);
      accumulate_cell(sum, own && i < h + 2, before.r, before.U, Fx, Fy, before.jx, before.jy);
    }
    before = now;
  };
#pragma unroll 1
  for (int i = 0; i < n; i += 2) {
    iteration(i, P);
    iteration(i + 1, Q);
  }
}

// What a workgroup reads: wide lattices below 4 GiB and above it, narrow ones below and above.
enum { kObsWhole, kObsBig, kObsColumns, kObsColumnsBig };

// Tiles blockIdx.x, blockIdx.x + blocks, ... of one lattice into one partial.
template <typename T, int EOS, int FORM>
__device__ __forceinline__ void obs_block(const T* __restrict__ f, const Geometry& geo, const DevC<double>& c,
                                          const ObsTiles& t, int block, int blocks, double* __restrict__ out) {
  __shared__ double2 ring[4][kRedThreads];
  __shared__ double sh[kNumRed][kRedThreads];
  ObsSum s{0.0, 0.0, 0.0, INFINITY, -INFINITY, 0.0, 0.0, 0u, 0u};
  for (int k = block; k < t.tiles; k += blocks) {
    if constexpr (FORM == kObsColumns) {
      obs_tile_narrow<T, EOS, unsigned>(f, geo, c, k * t.rows * t.groups, t.rows, t.groups, s, ring);
    } else if constexpr (FORM == kObsColumnsBig) {
      obs_tile_narrow<T, EOS, unsigned long long>(f, geo, c, k * t.rows * t.groups, t.rows, t.groups, s, ring);
    } else {
      const int rb = k / t.strips, y0 = rb * t.rows;
      obs_tile<T, EOS, FORM == kObsBig>(f, geo, c, (k - rb * t.strips) * kObsWidth, y0, min(t.rows, geo.ny - y0), s,
                                        ring);
    }
  }
  const double acc[kNumRed] = {s.mass, s.mx, s.my, s.lo, s.hi, s.v2, (double)s.n_domain, (double)s.n_bad};
  block_reduce_store(acc, sh, out);
}

template <typename T, int EOS, int FORM>
__global__ void __launch_bounds__(kRedThreads)
    k_obs(const T* __restrict__ f, const Geometry geo, const DevC<double> c, const ObsTiles t,
          double* __restrict__ partials) {
  obs_block<T, EOS, FORM>(f, geo, c, t, xcd_remap(blockIdx.x, gridDim.x), gridDim.x,
                    partials + (long long)xcd_remap(blockIdx.x, gridDim.x) * kNumRed);
}

// The partials of one lattice in a fixed order, and rho at the two sample cells
// of the Laplace measurement, (nx/2, ny/2) and (0, 0): kNumObs values.
template <typename T>
__device__ __forceinline__ void obs_finish(const T* __restrict__ f, const Geometry& geo,
                                           const double* __restrict__ partials, int nparts, double* __restrict__ red) {
  __shared__ double sh[kNumRed][kRedThreads];
  double acc[kNumRed] = {0.0, 0.0, 0.0, INFINITY, -INFINITY, 0.0, 0.0, 0.0};
#pragma unroll 4
  for (int b = threadIdx.x; b < nparts; b += kRedThreads) {
    const double* p = partials + (long long)b * kNumRed;
    acc[0] += p[0];
    acc[1] += p[1];
    acc[2] += p[2];
    acc[3] = fmin(acc[3], p[3]);
    acc[4] = fmax(acc[4], p[4]);
    acc[5] = fmax(acc[5], p[5]);
    acc[6] += p[6];
    acc[7] += p[7];
  }
  if (threadIdx.x < 2)
    red[kNumRed + threadIdx.x] = threadIdx.x == 0 ? cell_density(f, geo, geo.nx / 2, geo.ny / 2) : cell_density(f, geo, 0, 0);
  block_reduce_store(acc, sh, red);
}

template <typename T>
__global__ void __launch_bounds__(kRedThreads)
    k_obs_finish(const T* __restrict__ f, const Geometry geo, const double* __restrict__ partials, int nparts,
                 double* __restrict__ red) {
  obs_finish(f, geo, partials, nparts, red);
}

// A batch: one workgroup per partial of every domain, from a list, so that the
// workspace and the launch grow with the sum over the domains (one 4096^2 among
// 10,000 of 64^2: 10 MB; records for n times the largest would take 1.1 GB and 18
// million workgroups).  A domain has the tiles of the same lattice alone, so its
// observables are those of the lattice bit for bit and do not depend on what else
// is in the batch.  (Tiles of 16 rows where the batch is
// large read fewer rows twice, a call over 256 domains of 64^2 to 512^2 340 us
// against 393, and add them in another order.)
struct ObsDomain {
  Geometry g;
  DevC<double> c;
  const void* f[2];
  ObsTiles t;
  long long first;  // its partials in the batch's: first .. first + parts
  int parts;
};

struct ObsBlock {
  int domain, part;
};

template <typename T, int EOS, int FORM>
__global__ void __launch_bounds__(kRedThreads)
    k_batch_obs(const ObsDomain* __restrict__ dom, const ObsBlock* __restrict__ list, int parity,
                double* __restrict__ partials) {
  const ObsBlock b = list[blockIdx.x];
  const ObsDomain& D = dom[b.domain];
  obs_block<T, EOS, FORM>(static_cast<const T*>(D.f[parity]), D.g, D.c, D.t, b.part, D.parts,
                           partials + (D.first + b.part) * kNumRed);
}

template <typename T>
__global__ void __launch_bounds__(kRedThreads)
    k_batch_obs_finish(const ObsDomain* __restrict__ dom, int parity, const double* __restrict__ partials,
                       double* __restrict__ red) {
  const ObsDomain& D = dom[blockIdx.x];
  obs_finish(static_cast<const T*>(D.f[parity]), D.g, partials + D.first * kNumRed, D.parts,
             red + (long long)blockIdx.x * kNumObs);
}

template <typename T>
__global__ void k_plane_to_f64(const T* __restrict__ f, const Geometry geo, int a,
                               double* __restrict__ out) {
  const long long n = (long long)geo.nx * geo.ny;
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int y = (int)(i / geo.nx), x = (int)(i - (long long)y * geo.nx);
  out[i] = (double)f[state_index(geo, a, x, y)];
}

template <typename T>
__global__ void k_f64_to_plane(const double* __restrict__ in, const Geometry geo, int a,
                               T* __restrict__ f) {
  const long long n = (long long)geo.nx * geo.ny;
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int y = (int)(i / geo.nx), x = (int)(i - (long long)y * geo.nx);
  f[state_index(geo, a, x, y)] = T(in[i]);
}

static dim3 cells_grid(const Geometry& g) {
  const long long n = (long long)g.nx * g.ny;
  return dim3((unsigned)((n + 255) / 256));
}

int obs_partials_count(const Geometry& g) {
  const int tiles = obs_tiles(g).tiles;
  return tiles < kObsMaxBlocks ? tiles : kObsMaxBlocks;
}

hipError_t launch_plane_to_f64(lbm_precision prec, const Geometry& g, const void* f, int a,
                               double* out, hipStream_t s) {
  if (prec == LBM_FP32)
    hipLaunchKernelGGL(k_plane_to_f64<float>, cells_grid(g), dim3(256), 0, s,
                       static_cast<const float*>(f), g, a, out);
  else
    hipLaunchKernelGGL(k_plane_to_f64<double>, cells_grid(g), dim3(256), 0, s,
                       static_cast<const double*>(f), g, a, out);
  return hipGetLastError();
}

hipError_t launch_f64_to_plane(lbm_precision prec, const Geometry& g, const double* in, int a,
                               void* f, hipStream_t s) {
  if (prec == LBM_FP32)
    hipLaunchKernelGGL(k_f64_to_plane<float>, cells_grid(g), dim3(256), 0, s, in, g, a,
                       static_cast<float*>(f));
  else
    hipLaunchKernelGGL(k_f64_to_plane<double>, cells_grid(g), dim3(256), 0, s, in, g, a,
                       static_cast<double*>(f));
  return hipGetLastError();
}

template <typename T, int EOS>
static void density_t(const Geometry& g, const DevC<double>& c, const void* f, double* work,
                      hipStream_t s) {
  hipLaunchKernelGGL((k_density_fields<T, EOS>), cells_grid(g), dim3(256), 0, s,
                     static_cast<const T*>(f), g, c, work);
}

template <typename T>
static hipError_t density_p(const Geometry& g, const ModelConsts& m, const void* f, double* work,
                            hipStream_t s) {
  const DevC<double> c = make_devc<double>(m);
  switch (m.eos) {
    case LBM_EOS_IDEAL: density_t<T, LBM_EOS_IDEAL>(g, c, f, work, s); break;
    case LBM_EOS_CS: density_t<T, LBM_EOS_CS>(g, c, f, work, s); break;
    case LBM_EOS_VDW: density_t<T, LBM_EOS_VDW>(g, c, f, work, s); break;
    case LBM_EOS_PR: density_t<T, LBM_EOS_PR>(g, c, f, work, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_density_fields(lbm_precision prec, const Geometry& g, const ModelConsts& m,
                                 const void* f, double* work, hipStream_t s) {
  if (prec == LBM_FP32) return density_p<float>(g, m, f, work, s);
  return density_p<double>(g, m, f, work, s);
}

hipError_t launch_density(lbm_precision prec, const Geometry& g, const void* f, double* out, hipStream_t s) {
  if (prec == LBM_FP32)
    hipLaunchKernelGGL(k_density<float>, cells_grid(g), dim3(256), 0, s, static_cast<const float*>(f), g, out);
  else
    hipLaunchKernelGGL(k_density<double>, cells_grid(g), dim3(256), 0, s, static_cast<const double*>(f), g, out);
  return hipGetLastError();
}

hipError_t launch_velocity_field(lbm_precision prec, const Geometry& g, const ModelConsts& m,
                                 const void* f, const double* work, int comp, double* out,
                                 hipStream_t s) {
  const DevC<double> c = make_devc<double>(m);
  if (prec == LBM_FP32)
    hipLaunchKernelGGL(k_velocity<float>, cells_grid(g), dim3(256), 0, s,
                       static_cast<const float*>(f), g, c, work, comp, out);
  else
    hipLaunchKernelGGL(k_velocity<double>, cells_grid(g), dim3(256), 0, s,
                       static_cast<const double*>(f), g, c, work, comp, out);
  return hipGetLastError();
}

template <typename T, int EOS>
static hipError_t observables_e(const Geometry& g, const DevC<double>& c, const T* f, double* partials, double* red,
                                hipStream_t s) {
  const ObsTiles t = obs_tiles(g);
  const int np = obs_partials_count(g);
  const bool big = (unsigned long long)g.ny * g.row * sizeof(T) >= (1ull << 32);
  if (t.groups > 1 && big)
    hipLaunchKernelGGL((k_obs<T, EOS, kObsColumnsBig>), dim3(np), dim3(kRedThreads), 0, s, f, g, c, t, partials);
  else if (t.groups > 1)
    hipLaunchKernelGGL((k_obs<T, EOS, kObsColumns>), dim3(np), dim3(kRedThreads), 0, s, f, g, c, t, partials);
  else if (!big)
    hipLaunchKernelGGL((k_obs<T, EOS, kObsWhole>), dim3(np), dim3(kRedThreads), 0, s, f, g, c, t, partials);
  else
    hipLaunchKernelGGL((k_obs<T, EOS, kObsBig>), dim3(np), dim3(kRedThreads), 0, s, f, g, c, t, partials);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_obs_finish<T>, dim3(1), dim3(kRedThreads), 0, s, f, g, partials, np, red);
  return hipGetLastError();
}

template <typename T>
static hipError_t observables_t(const Geometry& g, const ModelConsts& m, const void* fv, double* partials, double* red,
                                hipStream_t s) {
  const DevC<double> c = make_devc<double>(m);
  const T* f = static_cast<const T*>(fv);
  switch (m.eos) {
    case LBM_EOS_IDEAL: return observables_e<T, LBM_EOS_IDEAL>(g, c, f, partials, red, s);
    case LBM_EOS_CS: return observables_e<T, LBM_EOS_CS>(g, c, f, partials, red, s);
    case LBM_EOS_VDW: return observables_e<T, LBM_EOS_VDW>(g, c, f, partials, red, s);
    case LBM_EOS_PR: return observables_e<T, LBM_EOS_PR>(g, c, f, partials, red, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_observables(lbm_precision prec, const Geometry& g, const ModelConsts& m, const void* f,
                              double* partials, double* red, hipStream_t s) {
  if (prec == LBM_FP32) return observables_t<float>(g, m, f, partials, red, s);
  return observables_t<double>(g, m, f, partials, red, s);
}

size_t obs_domain_bytes() { return sizeof(ObsDomain); }

size_t obs_block_bytes() { return sizeof(ObsBlock); }

void obs_fill_domain(const Geometry& g, const ModelConsts& m, const void* fa, const void* fb, long long first,
                     void* out) {
  *static_cast<ObsDomain*>(out) =
      ObsDomain{g, make_devc<double>(m), {fa, fb}, obs_tiles(g), first, obs_partials_count(g)};
}

void obs_fill_block(int domain, int part, void* out) { *static_cast<ObsBlock*>(out) = ObsBlock{domain, part}; }

bool obs_narrow(const Geometry& g) { return obs_tiles(g).groups > 1; }

template <typename T, int FORM>
static hipError_t batch_partials(int eos, const ObsBatch& q, const void* list, long long parts, int parity,
                                 hipStream_t s) {
  constexpr long long kMost = 1ll << 22;  // workgroups of a launch: its lanes are counted in 32 bits
  const ObsDomain* d = static_cast<const ObsDomain*>(q.domains);
  const dim3 block(kRedThreads);
  for (long long first = 0; first < parts; first += kMost) {
    const ObsBlock* l = static_cast<const ObsBlock*>(list) + first;
    const dim3 grid((unsigned)(parts - first < kMost ? parts - first : kMost));
    switch (eos) {
      case LBM_EOS_IDEAL: hipLaunchKernelGGL((k_batch_obs<T, LBM_EOS_IDEAL, FORM>), grid, block, 0, s, d, l, parity, q.partials); break;
      case LBM_EOS_CS: hipLaunchKernelGGL((k_batch_obs<T, LBM_EOS_CS, FORM>), grid, block, 0, s, d, l, parity, q.partials); break;
      case LBM_EOS_VDW: hipLaunchKernelGGL((k_batch_obs<T, LBM_EOS_VDW, FORM>), grid, block, 0, s, d, l, parity, q.partials); break;
      case LBM_EOS_PR: hipLaunchKernelGGL((k_batch_obs<T, LBM_EOS_PR, FORM>), grid, block, 0, s, d, l, parity, q.partials); break;
      default: return hipErrorInvalidValue;
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <typename T>
static hipError_t batch_observables_t(int eos, const ObsBatch& q, int parity, hipStream_t s) {
  hipError_t e = batch_partials<T, kObsWhole>(eos, q, q.list, q.wide, parity, s);
  if (e == hipSuccess)
    e = batch_partials<T, kObsColumns>(eos, q, static_cast<const ObsBlock*>(q.list) + q.wide, q.parts - q.wide, parity, s);
  constexpr long long kMost = 1ll << 22;
  for (long long first = 0; first < q.n && e == hipSuccess; first += kMost) {
    const dim3 grid((unsigned)(q.n - first < kMost ? q.n - first : kMost));
    hipLaunchKernelGGL(k_batch_obs_finish<T>, grid, dim3(kRedThreads), 0, s, static_cast<const ObsDomain*>(q.domains) + first,
                       parity, q.partials, q.red + first * kNumObs);
    e = hipGetLastError();
  }
  return e;
}

hipError_t launch_batch_observables(lbm_precision prec, int eos, const ObsBatch& q, int parity, hipStream_t s) {
  if (prec == LBM_FP32) return batch_observables_t<float>(eos, q, parity, s);
  return batch_observables_t<double>(eos, q, parity, s);
}

// ---------------------------------------------------------------------------
// Observables with no allocation: the partial sums live in one file-scope
// device array, resolved per device by hipGetSymbolAddress at a call's set-up.
// ---------------------------------------------------------------------------
constexpr size_t kNoAllocScratchDoubles = (size_t)kObsMaxBlocks * kNumRed + kNumObs;
static __device__ __align__(256) double scratch[kNoAllocScratchDoubles];

long long noalloc_max_cells() {
  return 1ll << 28;
}

hipError_t noalloc_scratch(double** out) {
  static std::mutex mu;
  static double* per_device[64] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!per_device[dev]) {
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    per_device[dev] = static_cast<double*>(ptr);
  }
  *out = per_device[dev];
  return hipSuccess;
}

}  // namespace lbm
