// k fused time steps of one block of a lattice, held in registers and LDS.
//
// The marching tiles (lbm_tile2.h) run a row at a time through a pipeline of
// 6 rows and 3 barriers a row, so a lattice too small to fill the GPU waits
// for a chain of H + 6 dependent rows however few cells it has.  Here a
// workgroup holds a whole block of w x h stored cells with its halo, up to C
// cells a lane, and every step is two phases over all of them at once:
//
//   density phase    pull f (step 1: from HBM, later steps: from the LDS
//                    planes), rho, U, psi                    -> LDS (U, psi)
//   collision phase  force, Q, collision                     -> LDS planes 1..8
//                    (last step: -> HBM; plane 0 stays in its register)
//
// with one barrier after each.  A step needs two more cells of halo on every
// side (one for the pull, one for the stencil), the first pull reads HBM
// directly, so k steps take a halo of m = 2k - 1 cells: the block computes
// W = w + 2m columns of H = h + 2m rows, numbered row by row over the lanes
// (any W, so a block divides its lattice evenly), and a cell at distance d
// from the block's rim takes part in the density phase of step s (from 0) if
// d >= 2s and in its collision if d >= 2s + 1; the stored cells are those
// with d >= m = 2(k - 1) + 1.  Neighbours of a cell that takes part are at
// most one cell nearer to the rim, so they took part in the phase before and
// lie inside the block.  The per-cell arithmetic is step_tile's, operation for
// operation: bitwise the states of single steps.
//
// What bounds it: on a lattice of one block a CU, the latency of a step's chain
// (about 0.7 us in FP32 and FP64) and a launch's 2 us, shared by its k
// steps: 100^2 FP64 1.55 us a step against 10.2 with the tiles, 300^2 FP32 2.2
// against 9.2.  On larger ones VALU issue, with the rim's recomputed cells as
// the overhead (1.3 collisions and 1.4 densities per cell stored and step at k = 3
// in 2,048-cell FP32 blocks), and the share of a block's loads and stores that no
// other workgroup's phases cover (a third to a half of a block's time by the model
// of lbm_plan.h): 1000 x 700 FP32 7.5 us a step against 11.9, 2048^2 35.6 against
// 39.9.  Register and LDS budget: FP32 blocks of 512 x 4 cells take 80 KB and 108
// VGPRs, so two workgroups a CU cover each other's loads and stores (one of
// 1024 x 4 in the whole LDS recomputes less and is 18% slower); 8 planes in LDS
// and not 9, since the rest population stays with its lane.  The first density
// and the last collision stand outside the step loop: inside it, with the
// choice of source and destination in branches, a lane moved its populations
// between registers 50 times a step and 100^2 FP64 took 1.9 us a step.
#pragma once

#include "lbm_tile.h"

namespace lbm {

// LDS of a block of up to B * C cells: (U, psi) and the planes 1..8 of each.
// The planes' stride is the capacity, not the block's cell count, so that
// every plane and every cell of a lane is an immediate offset of six addresses
// (rows -1, 0, +1 of the two arrays).
template <typename T, int B, int C>
struct BlockLds {
  typename V2<T>::t up[B * C];
  T F[8][B * C];
};

// The four neighbours' index steps of a cell in its block: to x - 1, x + 1,
// y - 1, y + 1.  Inside a halo they are -1, 1, -W, W for every cell; where the
// block is the whole periodic lattice they wrap, cell by cell.
struct Near {
  int l, r, s, n;
};

template <typename T>
__device__ __forceinline__ void block_stencil(const typename V2<T>::t* __restrict__ up, int i, const Near& d,
                                              T (&Un)[9], T (&Pn)[9]) {
  typename V2<T>::t v;
  v = up[i];               Un[0] = v.x; Pn[0] = v.y;
  v = up[i + d.r];         Un[1] = v.x; Pn[1] = v.y;  // ( 1, 0)
  v = up[(i + d.n)];       Un[2] = v.x; Pn[2] = v.y;  // ( 0, 1)
  v = up[i + d.l];         Un[3] = v.x; Pn[3] = v.y;  // (-1, 0)
  v = up[(i + d.s)];       Un[4] = v.x; Pn[4] = v.y;  // ( 0,-1)
  v = up[(i + d.n) + d.r]; Un[5] = v.x; Pn[5] = v.y;  // ( 1, 1)
  v = up[(i + d.n) + d.l]; Un[6] = v.x; Pn[6] = v.y;  // (-1, 1)
  v = up[(i + d.s) + d.l]; Un[7] = v.x; Pn[7] = v.y;  // (-1,-1)
  v = up[(i + d.s) + d.r]; Un[8] = v.x; Pn[8] = v.y;  // ( 1,-1)
}

// f_a(x - e_a) of planes 1..8 out of the LDS planes.
template <typename T, int N>
__device__ __forceinline__ void block_pull(const T (&F)[8][N], int i, const Near& d, T (&g)[9]) {
  g[1] = F[0][i + d.l];
  g[2] = F[1][(i + d.s)];
  g[3] = F[2][i + d.r];
  g[4] = F[3][(i + d.n)];
  g[5] = F[4][(i + d.s) + d.l];
  g[6] = F[5][(i + d.s) + d.r];
  g[7] = F[6][(i + d.n) + d.r];
  g[8] = F[7][(i + d.n) + d.l];
}

// Byte offsets of lattice cell (x, y)'s nine pulled populations, without the
// plane offset: row y + {0, -1, 1} and column x + {0, -1, 1} after the wrap.
struct CellAddr {
  unsigned c, w, e;     // columns x, x - 1, x + 1
  unsigned r, dn, up;   // rows y, y - 1, y + 1
};

template <typename T>
__device__ __forceinline__ CellAddr cell_addr(int x, int y, int nx, int ny, unsigned row_bytes) {
  CellAddr a;
  const unsigned sz = sizeof(T);
  a.c = x * sz;
  a.w = (x == 0 ? nx - 1 : x - 1) * sz;
  a.e = (x == nx - 1 ? 0 : x + 1) * sz;
  a.r = (unsigned)y * row_bytes;
  a.dn = y == 0 ? a.r + (unsigned)(ny - 1) * row_bytes : a.r - row_bytes;
  a.up = y == ny - 1 ? 0u : a.r + row_bytes;
  return a;
}

template <typename T>
__device__ __forceinline__ void block_gather(__amdgpu_buffer_rsrc_t f, const CellAddr& a, unsigned pb, T (&g)[9]) {
  g[0] = ld<T>(f, a.r + a.c, 0);
  g[1] = ld<T>(f, a.r + a.w, pb);
  g[2] = ld<T>(f, a.dn + a.c, 2 * pb);
  g[3] = ld<T>(f, a.r + a.e, 3 * pb);
  g[4] = ld<T>(f, a.up + a.c, 4 * pb);
  g[5] = ld<T>(f, a.dn + a.w, 5 * pb);
  g[6] = ld<T>(f, a.dn + a.e, 6 * pb);
  g[7] = ld<T>(f, a.up + a.e, 7 * pb);
  g[8] = ld<T>(f, a.up + a.w, 8 * pb);
}

// The phases of k steps over the block; lane t holds the cells t + j B.
// RIM: a cell takes part as long as its distance to the rim allows; otherwise
// the block is a whole periodic lattice and every cell always does.
template <typename T, int EOS, int B, int C, bool RIM>
__device__ __forceinline__ void block_steps(__amdgpu_buffer_rsrc_t out_buf, unsigned pb, const DevC<T>& c,
                                            int k, int W, T (&g)[C][9], const int (&dist)[C],
                                            const Near (&near)[C], const unsigned (&store_at)[C],
                                            BlockLds<T, B, C>& L) {
  using T2 = typename V2<T>::t;
  T rho[C];
  auto put_up = [&](int j, int i) {
    rho[j] = density(g[j]);
    L.up[i] = potentials<EOS>(rho[j], c);
  };
  auto collide = [&](int j, int i, T(&out)[9]) {
    T Un[9], Pn[9];
    block_stencil<T>(L.up, i, RIM ? Near{-1, 1, -W, W} : near[j], Un, Pn);
    collide_cell(g[j], rho[j], Un, Pn, c, out);
  };
#pragma unroll
  for (int j = 0; j < C; ++j)
    if (dist[j] >= 0) put_up(j, threadIdx.x + j * B);
  __syncthreads();
#pragma unroll 1
  for (int s = 1; s < k; ++s) {
#pragma unroll
    for (int j = 0; j < C; ++j) {
      const int i = threadIdx.x + j * B;
      if (dist[j] >= (RIM ? 2 * s - 1 : 0)) {
        T out[9];
        collide(j, i, out);
        g[j][0] = out[0];
#pragma unroll
        for (int a = 1; a < 9; ++a) L.F[a - 1][i] = out[a];
      }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < C; ++j) {
      const int i = threadIdx.x + j * B;
      if (dist[j] >= (RIM ? 2 * s : 0)) {
        block_pull(L.F, i, RIM ? Near{-1, 1, -W, W} : near[j], g[j]);
        put_up(j, i);
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int j = 0; j < C; ++j) {
    if (dist[j] >= (RIM ? 2 * k - 1 : 0)) {
      T out[9];
      collide(j, threadIdx.x + j * B, out);
#pragma unroll
      for (int a = 0; a < 9; ++a) st<T>(out_buf, store_at[j], a * pb, out[a]);
    }
  }
}

// One block: columns [x0, x0 + w) x rows [y0, y0 + h) advanced k steps;
// (w + 2m)(h + 2m) <= B C cells, m = 2k - 1.
template <typename T, int EOS, int B, int C>
__device__ __forceinline__ void block_tile(const T* __restrict__ fa, T* __restrict__ fb, const Geometry& geo,
                                           const DevC<T>& c, int x0, int y0, int w, int h, int k,
                                           BlockLds<T, B, C>& L) {
  const int nx = geo.nx, ny = geo.ny, m = 2 * k - 1, W = w + 2 * m, H = h + 2 * m, n = W * H;
  const unsigned pb = geo.pitch * sizeof(T), rb = (unsigned)(geo.row * sizeof(T));
  const unsigned total = (unsigned)((unsigned long long)geo.ny * geo.row * sizeof(T));
  const __amdgpu_buffer_rsrc_t ra = plane_rsrc(fa, total), rw = plane_rsrc(fb, total);
  // i / W for 0 <= i < 4096 and 3 <= W <= 4096, exactly: (i + 1/2) / W is at
  // least 1 / (2 W) away from any integer and the product rounds by less
  // than 2^-22 of itself, at most i / W * 2^-22 < 1 / (4 W)
  const float inv = 1.0f / (float)W;
  const bool far = m + 1 > nx || m + 1 > ny;  // the halo wraps more than once
  T g[C][9];
  int dist[C];
  Near near[C];
  unsigned store_at[C];
#pragma unroll
  for (int j = 0; j < C; ++j) {
    const int i = threadIdx.x + j * B;
    dist[j] = -1;
    store_at[j] = 0;
    if (i < n) {
      const int by = (int)(((float)i + 0.5f) * inv), bx = i - by * W;
      dist[j] = min(min(bx, W - 1 - bx), min(by, H - 1 - by));
      int x = x0 - m + bx, y = y0 - m + by;
      if (far) {
        x = (x % nx + nx) % nx;
        y = (y % ny + ny) % ny;
      } else {
        x = wrap_(x, nx);
        y = wrap_(y, ny);
      }
      const CellAddr a = cell_addr<T>(x, y, nx, ny, rb);
      store_at[j] = a.r + a.c;
      block_gather<T>(ra, a, pb, g[j]);
    }
  }
  block_steps<T, EOS, B, C, true>(rw, pb, c, k, W, g, dist, near, store_at, L);
}

// A whole periodic lattice of at most B C cells advanced k steps in one
// workgroup: no halo, neighbours by wrapped index.
template <typename T, int EOS, int B, int C>
__device__ __forceinline__ void block_lattice(const T* __restrict__ fa, T* __restrict__ fb, const Geometry& geo,
                                              const DevC<T>& c, int k, BlockLds<T, B, C>& L) {
  const int nx = geo.nx, ny = geo.ny, n = nx * ny;
  const unsigned pb = geo.pitch * sizeof(T), rb = (unsigned)(geo.row * sizeof(T));
  const unsigned total = (unsigned)((unsigned long long)geo.ny * geo.row * sizeof(T));
  const __amdgpu_buffer_rsrc_t ra = plane_rsrc(fa, total), rw = plane_rsrc(fb, total);
  T g[C][9];
  int dist[C];
  Near near[C];
  unsigned store_at[C];
#pragma unroll
  for (int j = 0; j < C; ++j) {
    const int i = threadIdx.x + j * B;
    dist[j] = -1;
    near[j] = Near{0, 0, 0, 0};
    store_at[j] = 0;
    if (i < n) {
      const int y = i / nx, x = i - y * nx;
      dist[j] = 0;
      near[j] = Near{x == 0 ? nx - 1 : -1, x == nx - 1 ? 1 - nx : 1, y == 0 ? n - nx : -nx,
                     y == ny - 1 ? nx - n : nx};
      const CellAddr a = cell_addr<T>(x, y, nx, ny, rb);
      store_at[j] = a.r + a.c;
      block_gather<T>(ra, a, pb, g[j]);
    }
  }
  block_steps<T, EOS, B, C, false>(rw, pb, c, k, 0, g, dist, near, store_at, L);
}

}  // namespace lbm
