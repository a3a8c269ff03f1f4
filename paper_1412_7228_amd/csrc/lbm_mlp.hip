// Surrogate network for surface-tension inversion: (A, kappa, T/Tc) -> (sigma,
// rho_l, rho_v), all normalised by the caller.  3 -> 128 -> 128 -> 128 -> 3,
// tanh hidden layers, linear output.
//
// Weights are held as bfloat16 (rounded from an FP32 master copy after every
// Adam step) and expanded exactly to FP32; activations, biases and every
// accumulation are FP32.  All products with 128 terms, and the sums over a
// workgroup's 32 samples, run on the matrix cores (v_mfma_f32_16x16x4f32, whose
// result is bitwise that of a chain of FP32 FMAs in the order of the terms).
//
// A call's few hundred samples leave the GPU nearly idle, so what counts is the
// chain of one sample block and the number of launches.  Training takes two
// launches an iteration: k_mlp_sample (forward, loss gradient and backward of 16
// samples a workgroup, a 16 x 16 block of a layer per wave, the activations
// staying in LDS and going to HBM once) and k_mlp_update (a workgroup per 16 x 16
// block of a layer's gradient: the products over each 32 samples, their sum in
// order, Adam, the rounded weights; and the loss).  The FP32 matrix rate of one CU
// is 1.7 us per 32 x 128 x 128 product, so the products of 32 samples all on one
// CU (six of them) took 24 us for 295 samples; split so, k_mlp_sample takes 12.8
// (its four dependent layer products and three tanh in turn) and k_mlp_update 5.6.  The 128 x 128 weights are kept a second time in the order in which
// the lanes take them (pack_at), so that a wave loads its 16 columns of a layer
// as four 16-byte loads a lane; read from the parameters' own order, with one
// 2-byte load per term, the products waited on 25 of the 29 us of a forward pass.
#include <hip/hip_runtime.h>

#include "lbm_internal.h"

namespace lbm {

constexpr int kH = 128, kIn = 3, kOut = 3, kRows = 32;
constexpr int kBlockRows = 16, kThreads = 512;  // samples and lanes of a workgroup: eight blocks of 16 columns
constexpr int oW1 = 0, oB1 = oW1 + kH * kIn, oW2 = oB1 + kH, oB2 = oW2 + kH * kH;
constexpr int oW3 = oB2 + kH, oB3 = oW3 + kH * kH, oW4 = oB3 + kH, oB4 = oW4 + kOut * kH;
constexpr int kNP = oB4 + kOut;  // 33,923
static_assert(kNP == 33923, "parameter count");

constexpr int kPad = kH + 4;  // row stride of the LDS activations: lanes (row i, term kk) on bank 4 i + kk
static_assert(kPad * sizeof(float) % 16 == 0, "rows are read four values at a time");

typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float bfw(const unsigned short* __restrict__ w, int i) {
  return __uint_as_float((unsigned)w[i] << 16);
}

// bfloat16 of an FP32 value: round to nearest, ties to even.
__device__ __forceinline__ unsigned short to_bf16(float f) {
  const unsigned u = __float_as_uint(f);
  return (unsigned short)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}

// Operands of a 16 x 16 block, lane l: A(l % 16, k) and B(k, l % 16) for
// k = 4 s + l / 16, s = 0, 1, ...; accumulator register r of lane l holds
// (row, column) = (4 (l / 16) + r, l % 16).
template <int K, class FA, class FB>
__device__ __forceinline__ f32x4 mfma_16x16(FA a, FB b, f32x4 acc) {
  const int lane = threadIdx.x & 63, i = lane & 15, kk = lane >> 4;
  float ta[K / 4], tb[K / 4];
#pragma unroll
  for (int s = 0; s < K / 4; ++s) {
    ta[s] = a(i, 4 * s + kk);
    tb[s] = b(4 * s + kk, i);
  }
  __builtin_amdgcn_sched_barrier(0);  // the reads in flight together, as in layer_block
#pragma unroll
  for (int s = 0; s < K / 4; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(ta[s], tb[s], acc, 0, 0, 0);
  return acc;
}

// The packed rounded weights: four matrices (the forward products of layers 2
// and 3, the backward ones of layers 3 and 2) of eight blocks of 16 columns, a
// block lane by lane, a lane's 32 terms k = 4 s + lane / 16 in a row.
enum { kPackF2 = 0, kPackF3 = 1, kPackB3 = 2, kPackB2 = 3 };
constexpr int kPackMatrix = kH * kH;
constexpr int kPacked = 4 * kPackMatrix;
__device__ __forceinline__ int pack_at(int matrix, int k, int col) {
  const int lane = (k & 3) * 16 + (col & 15);
  return ((matrix * 8 + (col >> 4)) * 64 + lane) * 32 + (k >> 2);
}

// Stores the rounded parameter i where the kernels read it.
__device__ __forceinline__ void put_weight(unsigned short* __restrict__ wb, unsigned short* __restrict__ wp, int i,
                                           float value) {
  const unsigned short h = to_bf16(value);
  wb[i] = h;
  // W[o][k] of layer 2 or 3: forward term k of column o, backward term o of column k
  if (i >= oW2 && i < oB2) {
    const int e = i - oW2, o = e / kH, k = e % kH;
    wp[pack_at(kPackF2, k, o)] = h;
    wp[pack_at(kPackB2, o, k)] = h;
  } else if (i >= oW3 && i < oB3) {
    const int e = i - oW3, o = e / kH, k = e % kH;
    wp[pack_at(kPackF3, k, o)] = h;
    wp[pack_at(kPackB3, o, k)] = h;
  }
}

// A wave's 16 columns of a packed matrix: 32 bfloat16 terms a lane.
struct Cols {
  uint4 v[4];
  __device__ __forceinline__ void load(const unsigned short* __restrict__ wp, int matrix, int block) {
    const uint4* p = reinterpret_cast<const uint4*>(wp + ((matrix * 8 + block) * 64 + (threadIdx.x & 63)) * 32);
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = p[q];
  }
  __device__ __forceinline__ float term(int s) const {  // s a compile-time constant after unrolling
    const uint4 q = v[s >> 3];
    const int w = (s >> 1) & 3;
    const unsigned u = w == 0 ? q.x : w == 1 ? q.y : w == 2 ? q.z : q.w;
    return __uint_as_float((s & 1) ? (u & 0xFFFF0000u) : (u << 16));
  }
};

// sum_k in[row][k] B(k, column) of one 16 x 16 block, B a wave's packed columns.
__device__ __forceinline__ f32x4 layer_block(const float (*in)[kPad], int row0, const Cols& w) {
  const int lane = threadIdx.x & 63, i = lane & 15, kk = lane >> 4;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  float a[kH / 4];
#pragma unroll
  for (int s = 0; s < kH / 4; ++s) a[s] = in[row0 + i][4 * s + kk];
  // all reads in flight before the chain starts: left to itself the compiler
  // reads two terms, waits for the LDS, multiplies and reads the next two
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int s = 0; s < kH / 4; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s], w.term(s), acc, 0, 0, 0);
  return acc;
}

// A lane's column of the first layer.
struct FirstCol {
  float w[kIn], b;
  __device__ __forceinline__ void load(const float* __restrict__ master, const unsigned short* __restrict__ wb) {
    const int o = threadIdx.x % kH;
#pragma unroll
    for (int k = 0; k < kIn; ++k) w[k] = bfw(wb, oW1 + o * kIn + k);
    b = master[oB1 + o];
  }
};

// h1 of 16 samples, xs -> out, by all lanes; rows past `valid` are zero.
__device__ __forceinline__ void first_layer(const float (*xs)[kIn], const FirstCol& c, int valid, float (*out)[kPad]) {
  const int o = threadIdx.x % kH;
#pragma unroll
  for (int r = threadIdx.x / kH; r < kBlockRows; r += kThreads / kH) {
    float z = c.b;
#pragma unroll
    for (int k = 0; k < kIn; ++k) z += c.w[k] * xs[r][k];
    out[r][o] = r < valid ? tanhf(z) : 0.f;
  }
}

// One hidden layer's 16 x 16 block of this wave: out = tanh(in W^T + b).
__device__ __forceinline__ void hidden_layer(const float (*in)[kPad], int row0, int block, const Cols& w, float bias,
                                             int valid, float (*out)[kPad]) {
  const int lane = threadIdx.x & 63, i = lane & 15, kk = lane >> 4;
  const f32x4 acc = layer_block(in, row0, w);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int row = row0 + 4 * kk + r;
    out[row][16 * block + i] = row < valid ? tanhf(acc[r] + bias) : 0.f;
  }
}

// The output layer's 16 rows from row0, by one wave: ys[row][o] = b4 + W4 h3.
__device__ __forceinline__ void output_layer(const float (*h3)[kPad], int row0, const float (*w4)[kH],
                                             const float* __restrict__ master, float (*ys)[kOut]) {
  const int lane = threadIdx.x & 63, i = lane & 15, kk = lane >> 4;
  const float b = i < kOut ? master[oB4 + i] : 0.f;
  const f32x4 start = {b, b, b, b};
  const f32x4 acc = mfma_16x16<kH>([&](int m, int k) { return h3[row0 + m][k]; },
                                   [&](int k, int j) { return j < kOut ? w4[j][k] : 0.f; }, start);
  if (i < kOut) {
#pragma unroll
    for (int r = 0; r < 4; ++r) ys[row0 + 4 * kk + r][i] = acc[r];
  }
}

__device__ __forceinline__ void load_w4(const unsigned short* __restrict__ wb, float (*w4)[kH]) {
  if (threadIdx.x < kOut * kH) (&w4[0][0])[threadIdx.x] = bfw(wb, oW4 + threadIdx.x);
}

// ---------------------------------------------------------------------------
// Forward: y = W4 h3 + b4, h_l = tanh(W_l h_{l-1} + b_l), 16 samples at a time
// per workgroup of eight waves, the weights staying in registers.  x and y may
// be pinned host memory (each element is read or written once).
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(kThreads)
    k_mlp_forward(const float* __restrict__ x, int B, const float* __restrict__ master,
                  const unsigned short* __restrict__ wb, const unsigned short* __restrict__ wp, float* __restrict__ y) {
  __shared__ float hA[kBlockRows][kPad], hB[kBlockRows][kPad], w4[kOut][kH];
  __shared__ float xs[kBlockRows][kIn], ys[kBlockRows][kOut];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  FirstCol c1;  // the operands needed first are loaded first
  c1.load(master, wb);
  load_w4(wb, w4);
  Cols c2, c3;
  c2.load(wp, kPackF2, w);
  c3.load(wp, kPackF3, w);
  const float b2 = master[oB2 + 16 * w + (lane & 15)], b3 = master[oB3 + 16 * w + (lane & 15)];
  for (long long r0 = (long long)blockIdx.x * kBlockRows; r0 < B; r0 += (long long)gridDim.x * kBlockRows) {
    const int valid = B - r0 < kBlockRows ? (int)(B - r0) : kBlockRows;
    if (tid < kBlockRows * kIn) (&xs[0][0])[tid] = tid < valid * kIn ? x[r0 * kIn + tid] : 0.f;
    __syncthreads();
    first_layer(xs, c1, valid, hA);
    __syncthreads();
    hidden_layer(hA, 0, w, c2, b2, valid, hB);
    __syncthreads();
    hidden_layer(hB, 0, w, c3, b3, valid, hA);
    __syncthreads();
    if (w == 0) output_layer(hA, 0, w4, master, ys);
    __syncthreads();
    if (tid < valid * kOut) y[r0 * kOut + tid] = (&ys[0][0])[tid];
  }
}

// What the gradients of the parameters need of each sample, rows past the last
// sample of a group of 32 zero: h1, h2, h3 and the gradients dz1, dz2, dz3 at the
// pre-activations [rows][128], the output gradient and the input [rows][3].
struct Acts {
  float* base;
  long long rows;  // capacity, a multiple of kRows
  __device__ __forceinline__ float* h(int l) const { return base + (l - 1) * rows * kH; }
  __device__ __forceinline__ float* dz(int l) const { return base + (l + 2) * rows * kH; }
  __device__ __forceinline__ float* dy() const { return base + 6 * rows * kH; }
  __device__ __forceinline__ float* x() const { return dy() + rows * kOut; }
};

// ---------------------------------------------------------------------------
// Forward and backward of 16 samples into `acts` and, if dx is not null, the
// input gradient.  The output gradient is dy, or with `t` that of the mean
// squared error over B x 3 outputs, 2 (y - t) / (3 B), with y written to y_out.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(kThreads)
    k_mlp_sample(const float* __restrict__ x, const float* __restrict__ dy, const float* __restrict__ t, int B,
                 const float* __restrict__ master, const unsigned short* __restrict__ wb,
                 const unsigned short* __restrict__ wp, const Acts acts, float* __restrict__ dx,
                 float* __restrict__ y_out) {
  __shared__ alignas(16) float h[3][kBlockRows][kPad];    // h1, h2, h3
  __shared__ alignas(16) float dzs[2][kBlockRows][kPad];  // gradients at two layers' pre-activations
  __shared__ float w4[kOut][kH];
  __shared__ float xs[kBlockRows][kIn], ys[kBlockRows][kOut], dys[kBlockRows][kOut];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, i = lane & 15, kk = lane >> 4;
  const long long r0 = (long long)blockIdx.x * kBlockRows;
  const int valid = B - r0 < kBlockRows ? (B > r0 ? (int)(B - r0) : 0) : kBlockRows;
  FirstCol c1;  // the operands needed first are loaded first
  c1.load(master, wb);
  const float xv = tid < valid * kIn ? x[r0 * kIn + tid] : 0.f;
  load_w4(wb, w4);
  Cols f2, f3, g3, g2;
  f2.load(wp, kPackF2, w);
  f3.load(wp, kPackF3, w);
  g3.load(wp, kPackB3, w);
  g2.load(wp, kPackB2, w);
  const float b2 = master[oB2 + 16 * w + i], b3 = master[oB3 + 16 * w + i];
  if (tid < kBlockRows * kIn) {
    (&xs[0][0])[tid] = xv;
    acts.x()[r0 * kIn + tid] = xv;
  }
  // a layer's rows from LDS to HBM, four values a lane
  auto keep = [&](const float (*from)[kPad], float* to) {
    const int r = tid >> 5, c = (tid & 31) * 4;
    *reinterpret_cast<float4*>(to + (r0 + r) * kH + c) = *reinterpret_cast<const float4*>(&from[r][c]);
  };
  __syncthreads();
  first_layer(xs, c1, valid, h[0]);
  __syncthreads();
  hidden_layer(h[0], 0, w, f2, b2, valid, h[1]);
  keep(h[0], acts.h(1));
  __syncthreads();
  hidden_layer(h[1], 0, w, f3, b3, valid, h[2]);
  keep(h[1], acts.h(2));
  __syncthreads();
  if (t) {
    if (w == 0) output_layer(h[2], 0, w4, master, ys);
    __syncthreads();
  }
  keep(h[2], acts.h(3));
  if (tid < kBlockRows * kOut) {
    const long long e = r0 * kOut + tid;
    float g = 0.f;
    if (tid < valid * kOut) {
      if (t) {
        const float inv = 1.f / (float)(B * kOut);
        const float v = (&ys[0][0])[tid];
        const float d = v - t[e];
        g = 2.f * d * inv;
        y_out[e] = v;
      } else {
        g = dy[e];
      }
    }
    (&dys[0][0])[tid] = g;
    acts.dy()[e] = g;
  }
  __syncthreads();
  // dz3 = (dy W4) (1 - h3^2)
#pragma unroll
  for (int e = tid; e < kBlockRows * kH; e += kThreads) {
    const int r = e / kH, k = e % kH;
    float s = 0.f;
#pragma unroll
    for (int o = 0; o < kOut; ++o) s += dys[r][o] * w4[o][k];
    dzs[0][r][k] = s * (1.f - h[2][r][k] * h[2][r][k]);
  }
  __syncthreads();
  // dn[r][k] = (sum_o dz[r][o] W[o][k]) (1 - hs[r][k]^2), layers 3 and 2
  auto back = [&](const float (*dz)[kPad], const Cols& c, const float (*hs)[kPad], float (*dn)[kPad]) {
    const f32x4 acc = layer_block(dz, 0, c);
    const int col = 16 * w + i;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = 4 * kk + r;
      dn[row][col] = acc[r] * (1.f - hs[row][col] * hs[row][col]);
    }
  };
  back(dzs[0], g3, h[1], dzs[1]);
  keep(dzs[0], acts.dz(3));
  __syncthreads();
  back(dzs[1], g2, h[0], dzs[0]);
  keep(dzs[1], acts.dz(2));
  __syncthreads();
  keep(dzs[0], acts.dz(1));
  if (dx && w == 0) {  // dx = dz1 W1
    const f32x4 acc = mfma_16x16<kH>([&](int m, int o) { return dzs[0][m][o]; },
                                     [&](int o, int j) { return j < kIn ? bfw(wb, oW1 + o * kIn + j) : 0.f; },
                                     f32x4{0.f, 0.f, 0.f, 0.f});
    if (i < kIn) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (4 * kk + r < valid) dx[(r0 + 4 * kk + r) * kIn + i] = acc[r];
    }
  }
}

// One 16 x 16 block of a parameter matrix's gradient, sum_r a[r][row] b[r][col]:
// operands, how many rows and columns of the block exist, where its (0, 0) is
// among the parameters and the strides there.  b null: a sum of a alone (a bias).
struct GradBlock {
  const float *a, *b;
  int lda, ldb, rows, cols, at, row_stride;
};

constexpr int kGradBlocks = 64 + 64 + 8 + 8 + 3 * 8 + 1;  // W2, W3, W4, W1, b1..b3, b4

__device__ __forceinline__ GradBlock grad_block(int n, const Acts& q) {
  if (n < 128) {
    const int layer = n < 64 ? 2 : 3, ob = (n & 63) >> 3, kb = n & 7;
    return {q.dz(layer) + 16 * ob, q.h(layer - 1) + 16 * kb, kH, kH, 16, 16,
            (layer == 2 ? oW2 : oW3) + 16 * ob * kH + 16 * kb, kH};
  }
  n -= 128;
  if (n < 8) return {q.dy(), q.h(3) + 16 * n, kOut, kH, kOut, 16, oW4 + 16 * n, kH};
  n -= 8;
  if (n < 8) return {q.dz(1) + 16 * n, q.x(), kH, kIn, 16, kIn, oW1 + 16 * n * kIn, kIn};
  n -= 8;
  if (n < 24) {
    const int layer = 1 + (n >> 3), ob = n & 7;
    return {q.dz(layer) + 16 * ob, nullptr, kH, 0, 16, 1, (layer == 1 ? oB1 : layer == 2 ? oB2 : oB3) + 16 * ob, 1};
  }
  return {q.dy(), nullptr, kOut, 0, kOut, 1, oB4, 1};
}

// The gradient of this thread's element (row tid / 16, column tid % 16): the
// products over each group of 32 samples (a wave per group, sixteen groups a
// round), then the groups in their order.
__device__ __forceinline__ float grad_sum(const GradBlock& g, int groups) {
  __shared__ float part[16][256];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, i = lane & 15, kk = lane >> 4;
  const bool has_a = i < g.rows, has_b = g.b && i < g.cols;
  float s = 0.f;
  for (int g0 = 0; g0 < groups; g0 += 16) {
    const int n = groups - g0 < 16 ? groups - g0 : 16;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int grp = w + 4 * q;
      if (grp < n) {  // uniform in a wave
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        float a[kRows / 4], b[kRows / 4];
#pragma unroll
        for (int m = 0; m < kRows / 4; ++m) {
          const long long r = (long long)(g0 + grp) * kRows + 4 * m + kk;
          a[m] = has_a ? g.a[r * g.lda + i] : 0.f;
          b[m] = has_b ? g.b[r * g.ldb + i] : (!g.b && i == 0 ? 1.f : 0.f);
        }
#pragma unroll
        for (int m = 0; m < kRows / 4; ++m) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[m], b[m], acc, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) part[grp][(4 * kk + r) * 16 + i] = acc[r];
      }
    }
    __syncthreads();
    for (int q = 0; q < n; ++q) s += part[q][tid];
    __syncthreads();
  }
  return s;
}

__global__ void __launch_bounds__(256) k_mlp_gradient(const Acts acts, int B, float* __restrict__ grad) {
  const GradBlock g = grad_block(blockIdx.x, acts);
  const float s = grad_sum(g, (B + kRows - 1) / kRows);
  const int row = threadIdx.x >> 4, col = threadIdx.x & 15;
  if (row < g.rows && col < g.cols) grad[g.at + row * g.row_stride + col] = s;
}

// The gradients, Adam on the FP32 master parameters and their rounded copies;
// the last block instead adds up the mean squared error over B x 3 outputs into
// loss[0].
__global__ void __launch_bounds__(256)
    k_mlp_update(const Acts acts, float* __restrict__ p, float* __restrict__ m, float* __restrict__ v,
                 unsigned short* __restrict__ wb, unsigned short* __restrict__ wp, float lr, float b1, float b2,
                 float eps, float c1, float c2, const float* __restrict__ y, const float* __restrict__ t, int B,
                 float* __restrict__ loss) {
  if (blockIdx.x == kGradBlocks) {
    __shared__ float sh[256];
    const int n = B * kOut;
    const float inv = 1.f / (float)n;
    float s = 0.f;
#pragma unroll 4
    for (int i = threadIdx.x; i < n; i += 256) {
      const float d = y[i] - t[i];
      s += d * d;
    }
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
      if ((int)threadIdx.x < st) sh[threadIdx.x] += sh[threadIdx.x + st];
      __syncthreads();
    }
    if (threadIdx.x == 0) loss[0] = sh[0] * inv;
    return;
  }
  const GradBlock g = grad_block(blockIdx.x, acts);
  const int row = threadIdx.x >> 4, col = threadIdx.x & 15;
  const bool own = row < g.rows && col < g.cols;
  const int i = own ? g.at + row * g.row_stride + col : 0;
  const float m0 = m[i], v0 = v[i], p0 = p[i];  // in flight while the products run
  const float gi = grad_sum(g, (B + kRows - 1) / kRows);
  if (!own) return;
  const float mi = b1 * m0 + (1.f - b1) * gi;
  const float vi = b2 * v0 + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  const float pi = p0 - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  p[i] = pi;
  put_weight(wb, wp, i, pi);
}

__global__ void k_mlp_round(const float* __restrict__ p, unsigned short* __restrict__ wb,
                            unsigned short* __restrict__ wp) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < kNP) put_weight(wb, wp, i, p[i]);
}

__global__ void k_mlp_read(const float* __restrict__ p, float* __restrict__ out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < kNP) out[i] = p[i];
}

int mlp_param_count() { return kNP; }
int mlp_packed_count() { return kPacked; }

static long long acts_rows(int max_batch) { return (max_batch + kRows - 1) / kRows * (long long)kRows; }
size_t mlp_acts_bytes(int max_batch) { return (size_t)acts_rows(max_batch) * (6 * kH + kOut + kIn) * sizeof(float); }

hipError_t launch_mlp_forward(const float* x, int B, const MlpWeights& w, float* y, hipStream_t s) {
  const int blocks = (B + kBlockRows - 1) / kBlockRows;
  hipLaunchKernelGGL(k_mlp_forward, dim3(blocks < 1024 ? blocks : 1024), dim3(kThreads), 0, s, x, B, w.master,
                     w.rounded, w.packed, y);
  return hipGetLastError();
}

hipError_t launch_mlp_sample(const float* x, const float* dy, const float* t, int B, const MlpWeights& w, float* acts,
                             int max_batch, float* dx, float* y, hipStream_t s) {
  // whole groups of 32 samples: the rows past B are written as zeros
  const int blocks = (B + kRows - 1) / kRows * (kRows / kBlockRows);
  hipLaunchKernelGGL(k_mlp_sample, dim3(blocks), dim3(kThreads), 0, s, x, dy, t, B, w.master, w.rounded, w.packed,
                     Acts{acts, acts_rows(max_batch)}, dx, y);
  return hipGetLastError();
}

hipError_t launch_mlp_gradient(float* acts, int max_batch, int B, float* grad, hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_gradient, dim3(kGradBlocks), dim3(256), 0, s, Acts{acts, acts_rows(max_batch)}, B, grad);
  return hipGetLastError();
}

hipError_t launch_mlp_update(float* acts, int max_batch, const MlpWeights& w, float* m, float* v, float lr, float b1,
                             float b2, float eps, float c1, float c2, const float* y, const float* t, int B,
                             float* loss, hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_update, dim3(kGradBlocks + 1), dim3(256), 0, s, Acts{acts, acts_rows(max_batch)}, w.master,
                     m, v, w.rounded, w.packed, lr, b1, b2, eps, c1, c2, y, t, B, loss);
  return hipGetLastError();
}

hipError_t launch_mlp_read(const float* master, float* out, hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_read, dim3((kNP + 255) / 256), dim3(256), 0, s, master, out);
  return hipGetLastError();
}

hipError_t launch_mlp_round(const MlpWeights& w, hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_round, dim3((kNP + 255) / 256), dim3(256), 0, s, w.master, w.rounded, w.packed);
  return hipGetLastError();
}

}  // namespace lbm
