// Calibration surrogate: a 4 -> 128 -> 128 -> 128 -> 4 multilayer perceptron
// with GELU hidden activations (Hendrycks and Gimpel, 2016), mapping a
// calibration tuple (model, Tr, width parameter, kappa) to the equilibrium
// properties (rho_l, rho_v, surface tension, interface width), trained with
// Adam (Kingma and Ba, 2015) on equilibria computed by the batched lattices.
//
// Kernels (gfx950):
//   k_mlp_forward  tiles of 16 samples, one wavefront per 16 columns of a
//                  layer (eight per workgroup), the weights of its columns in
//                  registers for every tile the workgroup walks;
//   k_mlp_grad     forward, loss and back-propagation of a tile in one
//                  workgroup; a workgroup walks several tiles and accumulates
//                  its weight gradient in its own slice of the workspace;
//   k_mlp_reduce   sums the per-workgroup slices in a fixed order, so the
//                  gradient is deterministic; in a training step it also
//                  makes the Adam update;
//   k_mlp_adam     one elementwise Adam update.
// The network is ~34k parameters and a training batch a few hundred samples,
// so a step is bound by latency: the chain of layers, the memory round trips
// and the launches.  All weights a wavefront needs (forward and transposed)
// are therefore fetched at once when the kernel starts, and every contraction
// runs on the matrix cores (mfma blocks of 16 samples by 16 columns), with
// activations and errors passed through LDS between the layers.
//
// BF16 mode rounds every product operand (layer inputs and weights) to
// bfloat16, round to nearest even; products of two bfloat16 values are exact
// in FP32 and all sums accumulate in FP32: its two hidden layers run as
// v_mfma_f32_16x16x16_bf16.  Biases and back-propagated errors are not
// rounded, so the backward products, like FP32 mode's hidden layers, run as
// v_mfma_f32_16x16x4_f32, whose sum is the ascending chain of fused
// multiply-adds of its four products (the same bits as an fmaf loop); the
// weight rounding is treated as the identity in the gradient.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <mutex>

#include "lbm.h"

namespace mlpk {

constexpr int H = 128, NI = 4, NO = 4;
constexpr int OFF_W1 = 0;
constexpr int OFF_B1 = OFF_W1 + NI * H;
constexpr int OFF_W2 = OFF_B1 + H;
constexpr int OFF_B2 = OFF_W2 + H * H;
constexpr int OFF_W3 = OFF_B2 + H;
constexpr int OFF_B3 = OFF_W3 + H * H;
constexpr int OFF_W4 = OFF_B3 + H;
constexpr int OFF_B4 = OFF_W4 + H * NO;
constexpr int NPARAM = OFF_B4 + NO;
static_assert(NPARAM == LBM_MLP_NPARAMS, "parameter count");
constexpr int TS = 16;         // samples per tile
constexpr int NT = 512;        // threads per workgroup: wavefront w has the columns 16 w ..
constexpr int LP = H + 4;      // LDS row: 16 samples x 4 columns fall on 64 different banks
constexpr int MAX_GRAD_BLOCKS = 128;

struct Norm {
  float xs[NI], xk[NI], ys[NO], yk[NO];
};

__device__ __forceinline__ float bf16r(float v) {
  unsigned u = __float_as_uint(v);
  u = (u + 0x7FFFu + ((u >> 16) & 1u)) & 0xFFFF0000u;
  return __uint_as_float(u);
}

template <int BF>
__device__ __forceinline__ float rnd(float v) {
  if constexpr (BF) return bf16r(v);
  else return v;
}

__device__ __forceinline__ float gelu(float z) {
  return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f));
}

__device__ __forceinline__ float gelu_d(float z) {
  return 0.5f * (1.0f + erff(z * 0.70710678118654752f)) +
         z * expf(-0.5f * z * z) * 0.39894228040143268f;
}

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// Bit pattern of a float that is already a bfloat16 value (low half zero).
__device__ __forceinline__ short bf16_bits(float v) {
  return (short)(__float_as_uint(v) >> 16);
}

// Matrix-core blocks of 16 x 16 (lane l: r = l % 16, q = l / 16).
// v_mfma_f32_16x16x16_bf16: lane l supplies A[r][4 q + v] and B[4 q + v][r];
// v_mfma_f32_16x16x4_f32: A[r][q] and B[q][r]; both receive D[4 q + v][r]
// (v = 0..3).  A tile's rows are its samples, so lane l of wavefront w holds
// samples 4 q + v of column 16 w + r of every layer.
struct Lane {
  int r, q, j;  // j: the lane's column
  __device__ __forceinline__ Lane() {
    const int l = threadIdx.x & 63;
    r = l & 15;
    q = l >> 4;
    j = 16 * (threadIdx.x >> 6) + r;
  }
};

// Wait for a matrix-core result before it is used across a branch: the
// hardware needs 11 wait states from a 16x16x4 FP32 mfma to a store that reads
// its result, and the compiler counted none where a branch lay between the two
// (stores of stale values).
__device__ __forceinline__ void mfma_settle(f32x4& v) {
  asm volatile("s_nop 7\n\ts_nop 7" : "+v"(v));
}

// Orders a wavefront's LDS writes before the reads of its other lanes (no wait
// of its own: a wavefront's LDS accesses are served in order).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A 128 x 128 weight matrix as the workgroup fetches it: thread t has float4s
// t, t + NT, ... of its 4096, so that every access is a whole line (fetched in
// operand order, lane by lane, the two matrices took 17 us of a 28 us
// gradient); stage() rounds it into LDS, whose rows are LP long: the operands
// of the BF16 forward product (rows 4 q + v, columns r) and of the transposed
// one (rows r, columns 4 kk + q) then fall on 64 different banks.
constexpr int W4T = H * H / 4 / NT;
struct Mat {
  f32x4 w[W4T];
  __device__ __forceinline__ void fetch(const float* __restrict__ W) {
    if (((uintptr_t)W & 15) == 0) {
#pragma unroll
      for (int i = 0; i < W4T; ++i) w[i] = ((const f32x4*)W)[threadIdx.x + i * NT];
    } else {  // parameters that start inside a caller's larger buffer
#pragma unroll
      for (int i = 0; i < W4T; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) w[i][v] = W[4 * (threadIdx.x + i * NT) + v];
    }
  }
  template <int BF>
  __device__ __forceinline__ void stage(float (*s_w)[LP]) const {
#pragma unroll
    for (int i = 0; i < W4T; ++i) {
      const int e = threadIdx.x + i * NT;
      f32x4 x;
#pragma unroll
      for (int v = 0; v < 4; ++v) x[v] = rnd<BF>(w[i][v]);
      *(f32x4*)&s_w[e / (H / 4)][4 * (e % (H / 4))] = x;
    }
  }
};

// A hidden layer's staged weights for the wavefront's columns, in operand
// order, and the product a W + b of a tile with them.
template <int BF>
struct FwdW;
template <>
struct FwdW<1> {
  bf16x4 w[H / 16];
  __device__ __forceinline__ void read(const float (*s_w)[LP], const Lane& n) {
#pragma unroll
    for (int kb = 0; kb < H / 16; ++kb)
#pragma unroll
      for (int v = 0; v < 4; ++v) w[kb][v] = bf16_bits(s_w[kb * 16 + 4 * n.q + v][n.j]);
  }
  __device__ __forceinline__ f32x4 run(const float (*a)[LP], float b, const Lane& n) const {
    f32x4 acc = {b, b, b, b};
#pragma unroll
    for (int kb = 0; kb < H / 16; ++kb) {
      const f32x4 x = *(const f32x4*)&a[n.r][kb * 16 + 4 * n.q];
      bf16x4 av;
#pragma unroll
      for (int v = 0; v < 4; ++v) av[v] = bf16_bits(x[v]);
      acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(av, w[kb], acc, 0, 0, 0);
    }
    mfma_settle(acc);
    return acc;
  }
};
template <>
struct FwdW<0> {
  float w[H / 4];
  __device__ __forceinline__ void read(const float (*s_w)[LP], const Lane& n) {
#pragma unroll
    for (int kk = 0; kk < H / 4; ++kk) w[kk] = s_w[4 * kk + n.q][n.j];
  }
  __device__ __forceinline__ f32x4 run(const float (*a)[LP], float b, const Lane& n) const {
    f32x4 acc = {b, b, b, b};
#pragma unroll
    for (int kk = 0; kk < H / 4; ++kk)
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[n.r][4 * kk + n.q], w[kk], acc, 0, 0, 0);
    mfma_settle(acc);
    return acc;
  }
};

// The rest of a lane's forward weights: its column of the input layer, the
// biases of its columns (b4: of output r % NO).
template <int BF>
struct Net {
  float w1[NI], b1, b2, b3, b4;
  __device__ __forceinline__ void load(const float* __restrict__ P, const Lane& n) {
#pragma unroll
    for (int k = 0; k < NI; ++k) w1[k] = rnd<BF>(P[OFF_W1 + k * H + n.j]);
    b1 = P[OFF_B1 + n.j];
    b2 = P[OFF_B2 + n.j];
    b3 = P[OFF_B3 + n.j];
    b4 = P[OFF_B4 + (n.r & (NO - 1))];
  }
};

// The output layer's weights, rounded, into LDS (visible after a barrier).
template <int BF>
__device__ __forceinline__ void stage_w4(const float* __restrict__ P, float (*s_w4)[NO]) {
  s_w4[threadIdx.x / NO][threadIdx.x % NO] = rnd<BF>(P[OFF_W4 + threadIdx.x]);  // NT = H NO
}

// The layers of a tile's forward pass: z the lane's pre-activations (kept for
// the derivative), the rounded activations to LDS.  Sample rows without a
// sample hold zero inputs and finite values that the callers ignore.
template <int BF>
__device__ __forceinline__ void activate(const f32x4& z, const Lane& n, float (*a)[LP]) {
#pragma unroll
  for (int v = 0; v < 4; ++v) a[4 * n.q + v][n.j] = rnd<BF>(gelu(z[v]));
}

template <int BF>
__device__ __forceinline__ f32x4 input_layer(const Net<BF>& net, const Lane& n,
                                             const float (*s_a0)[NI]) {
  f32x4 z;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    float acc = net.b1;
#pragma unroll
    for (int k = 0; k < NI; ++k) acc = fmaf(net.w1[k], s_a0[4 * n.q + v][k], acc);
    z[v] = acc;
  }
  return z;
}

// Outputs in normalised log space, by wavefront 0 (visible to it; the others
// need a barrier).
__device__ __forceinline__ void output_layer(const float (*a)[LP], const float (*s_w4)[NO],
                                             float b4, const Lane& n, float (*s_o)[NO]) {
  if (threadIdx.x >= 64) return;
  // (columns r >= NO repeat the first ones and are dropped)
  f32x4 acc = {b4, b4, b4, b4};
#pragma unroll
  for (int kk = 0; kk < H / 4; ++kk)
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[n.r][4 * kk + n.q],
                                               s_w4[4 * kk + n.q][n.r & (NO - 1)], acc, 0, 0, 0);
  mfma_settle(acc);
  if (n.r < NO)
#pragma unroll
    for (int v = 0; v < 4; ++v) s_o[4 * n.q + v][n.r] = acc[v];
  wave_sync();
}

// Predictions, a workgroup walking tiles with a stride of the grid.  256
// samples (16 workgroups): 7.5 us (12.5 us with the weights read from L2 inside
// the products).
template <int BF>
__global__ __launch_bounds__(NT) void k_mlp_forward(const float* __restrict__ P, Norm nm,
                                                    const float* __restrict__ X, int n,
                                                    float* __restrict__ Y) {
  __shared__ float s_a0[TS][NI];
  __shared__ __attribute__((aligned(16))) float s_a[3][TS][LP];
  __shared__ __attribute__((aligned(16))) float s_w[H][LP];
  __shared__ float s_o[TS][NO], s_w4[H][NO];
  const int t = threadIdx.x;
  const Lane ln;
  FwdW<BF> l2, l3;
  Net<BF> net;
  {
    Mat m2, m3;
    m2.fetch(P + OFF_W2);
    m3.fetch(P + OFF_W3);
    net.load(P, ln);
    stage_w4<BF>(P, s_w4);
    m2.template stage<BF>(s_w);
    __syncthreads();
    l2.read(s_w, ln);
    __syncthreads();
    m3.template stage<BF>(s_w);
    __syncthreads();
    l3.read(s_w, ln);
  }
  const int ntiles = (n + TS - 1) / TS;
  for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const int s = t / NI, k = t % NI;
    const int row = tile * TS + s;
    if (t < TS * NI)
      s_a0[s][k] = row < n ? rnd<BF>((X[(size_t)row * NI + k] - nm.xs[k]) * nm.xk[k]) : 0.0f;
    __syncthreads();
    activate<BF>(input_layer(net, ln, s_a0), ln, s_a[0]);
    __syncthreads();
    activate<BF>(l2.run(s_a[0], net.b2, ln), ln, s_a[1]);
    __syncthreads();
    activate<BF>(l3.run(s_a[1], net.b3, ln), ln, s_a[2]);
    __syncthreads();
    output_layer(s_a[2], s_w4, net.b4, ln, s_o);
    if (t < TS * NO && row < n)  // wavefront 0, which wrote s_o (NI = NO)
      Y[(size_t)row * NO + k] = expf(s_o[s][k] * nm.yk[k] + nm.ys[k]);
    // (wavefront 0 alone writes s_a0 of the next tile before the next barrier,
    // and every wavefront has read this tile's before the last one)
  }
}

// Gradient slice update: the first tile of a workgroup stores, later tiles
// add.  Each slice element is owned by one thread in every phase, the same
// thread for every tile.
template <class V>
__device__ __forceinline__ void gput(V* p, V g, bool first) {
  if (first) *p = g;
  else *p += g;
}

// Weight gradient of a hidden layer, dW[k][j] = sum_s a[s][k] d[s][j] (the
// wavefront's columns j as the rows of the block, so that a lane gets four
// consecutive j of one k), and its bias gradient.
__device__ __forceinline__ void hidden_grad(const float (*a)[LP], const float (*d)[LP],
                                            const Lane& n, float* __restrict__ GW,
                                            float* __restrict__ GB, bool first) {
  const int jb = n.j - n.r;
  float dj[TS / 4], ak[H / 16][TS / 4];
#pragma unroll
  for (int ss = 0; ss < TS / 4; ++ss) {
    dj[ss] = d[4 * ss + n.q][n.j];
#pragma unroll
    for (int kb = 0; kb < H / 16; ++kb) ak[kb][ss] = a[4 * ss + n.q][16 * kb + n.r];
  }
  f32x4 g[H / 16];
#pragma unroll
  for (int kb = 0; kb < H / 16; ++kb) g[kb] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  // (the chains of the eight blocks interleaved: each waits for itself only)
#pragma unroll
  for (int ss = 0; ss < TS / 4; ++ss)
#pragma unroll
    for (int kb = 0; kb < H / 16; ++kb)
      g[kb] = __builtin_amdgcn_mfma_f32_16x16x4f32(dj[ss], ak[kb][ss], g[kb], 0, 0, 0);
  asm volatile("s_nop 7\n\ts_nop 7"  // mfma_settle of all eight
               : "+v"(g[0]), "+v"(g[1]), "+v"(g[2]), "+v"(g[3]), "+v"(g[4]), "+v"(g[5]),
                 "+v"(g[6]), "+v"(g[7]));
  static_assert(H / 16 == 8, "blocks settled");
#pragma unroll
  for (int kb = 0; kb < H / 16; ++kb) {
    gput((f32x4*)&GW[(16 * kb + n.r) * H + jb + 4 * n.q], g[kb], first);
  }
  if (threadIdx.x < H) {
    float b = 0.0f;
#pragma unroll
    for (int s = 0; s < TS; ++s) b += d[s][threadIdx.x];
    gput(&GB[threadIdx.x], b, first);
  }
}

// Transposed product of a hidden layer with staged weights: (d W^T)[s][k] for
// the wavefront's columns k.
__device__ __forceinline__ f32x4 hidden_back(const float (*d)[LP], const float (*s_w)[LP],
                                             const Lane& n) {
  f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int kk = 0; kk < H / 4; ++kk)
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(d[n.r][4 * kk + n.q], s_w[n.j][4 * kk + n.q], acc,
                                               0, 0, 0);
  mfma_settle(acc);
  return acc;
}

// Loss and gradient partials.  Workgroup g handles tiles g, g + G, ...
// (G <= number of tiles, so every workgroup has at least one); its gradient
// slice part[g * NPARAM ...] and loss partial lpart[g] are fully written by
// this kernel (no prior clearing needed).  256 samples (16 workgroups): 17 us
// (58 us with the backward products on the vector ALUs); four products of 2048
// cycles each on the FP32 matrix cores of one CU are 3.5 us of it, the rest
// the fetch of the weights and the chain of layers.
template <int BF>
__global__ __launch_bounds__(NT) void k_mlp_grad(const float* __restrict__ P, Norm nm,
                                                 const float* __restrict__ X,
                                                 const float* __restrict__ Y,
                                                 const int* __restrict__ idx, int n, int nrows,
                                                 float scale, float* __restrict__ part,
                                                 float* __restrict__ lpart) {
  __shared__ float s_a0[TS][NI];
  __shared__ __attribute__((aligned(16))) float s_a[3][TS][LP];
  __shared__ __attribute__((aligned(16))) float s_w[H][LP];
  __shared__ float s_d[TS][LP];   // dL/dz of layers 3 and 1
  __shared__ float s_e[TS][LP];   // dL/dz of layer 2
  __shared__ __attribute__((aligned(16))) float s_o[TS][NO];  // outputs, then dL/dout
  __shared__ __attribute__((aligned(16))) float s_w4[H][NO];
  __shared__ int s_bad;
  const int t = threadIdx.x;
  Lane ln;
  if (t == 0) s_bad = 0;
  Mat m2, m3;
  m2.fetch(P + OFF_W2);
  m3.fetch(P + OFF_W3);
  Net<BF> net;
  net.load(P, ln);
  stage_w4<BF>(P, s_w4);
  __syncthreads();
  float lacc = 0.0f;
  const int ntiles = (n + TS - 1) / TS;
  for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    // addresses formed anew for each tile: hoisted out of the loop they take
    // the registers that the weights are in
    asm volatile("" : "+v"(ln.r), "+v"(ln.q), "+v"(ln.j));
    int slice = blockIdx.x * NPARAM;
    asm volatile("" : "+s"(slice));
    float* const G = part + slice;
    const bool first = tile == (int)blockIdx.x;
    // wavefront 0: input k and target k of sample s (NI = NO)
    const int s = t / NI, k = t % NI;
    bool valid = false;
    float yv = 1.0f;
    if (t < TS * NI) {
      float v = 0.0f;
      if (tile * TS + s < n) {
        const int r = idx ? idx[tile * TS + s] : tile * TS + s;
        if (r >= 0 && r < nrows) {
          valid = true;
          v = rnd<BF>((X[(size_t)r * NI + k] - nm.xs[k]) * nm.xk[k]);
          yv = Y[(size_t)r * NO + k];
        } else {
          s_bad = 1;
        }
      }
      s_a0[s][k] = v;
    }
    m2.template stage<BF>(s_w);
    __syncthreads();
    f32x4 z[3];
    FwdW<BF> lw;
    lw.read(s_w, ln);
    z[0] = input_layer(net, ln, s_a0);
    activate<BF>(z[0], ln, s_a[0]);
    __syncthreads();
    m3.template stage<BF>(s_w);
    z[1] = lw.run(s_a[0], net.b2, ln);
    activate<BF>(z[1], ln, s_a[1]);
    __syncthreads();
    lw.read(s_w, ln);
    z[2] = lw.run(s_a[1], net.b3, ln);
    activate<BF>(z[2], ln, s_a[2]);
    __syncthreads();
    output_layer(s_a[2], s_w4, net.b4, ln, s_o);
    // loss and dL/dout (zero for padding rows and rejected indices), by
    // wavefront 0, which wrote the outputs
    if (t < TS * NO) {
      float dv = 0.0f;
      if (valid) {
        const float tgt = (logf(yv) - nm.ys[k]) / nm.yk[k];
        const float res = s_o[s][k] - tgt;
        lacc = fmaf(res, res, lacc);
        dv = 2.0f * res * scale;
      }
      s_o[s][k] = dv;
    }
    __syncthreads();
    // output layer: dW4[k][o] = sum_s a3[s][k] dout[s][o]
    {
      const f32x4 w4 = *(const f32x4*)s_w4[ln.j];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const f32x4 dv = *(const f32x4*)s_o[4 * ln.q + v];
        float da = 0.0f;
#pragma unroll
        for (int o = 0; o < NO; ++o) da = fmaf(dv[o], w4[o], da);
        s_d[4 * ln.q + v][ln.j] = da * gelu_d(z[2][v]);
      }
      float g = 0.0f;  // NT = H NO elements
#pragma unroll
      for (int i = 0; i < TS; ++i) g = fmaf(s_a[2][i][t / NO], s_o[i][t % NO], g);
      gput(&G[OFF_W4 + t], g, first);
      if (t < NO) {
        float b = 0.0f;
#pragma unroll
        for (int i = 0; i < TS; ++i) b += s_o[i][t];
        gput(&G[OFF_B4 + t], b, first);
      }
    }
    __syncthreads();
    // hidden layers 3 and 2
    {
      const f32x4 e = hidden_back(s_d, s_w, ln);
#pragma unroll
      for (int v = 0; v < 4; ++v) s_e[4 * ln.q + v][ln.j] = e[v] * gelu_d(z[1][v]);
      hidden_grad(s_a[1], s_d, ln, G + OFF_W3, G + OFF_B3, first);
    }
    __syncthreads();
    m2.template stage<BF>(s_w);
    __syncthreads();
    {
      const f32x4 e = hidden_back(s_e, s_w, ln);
#pragma unroll
      for (int v = 0; v < 4; ++v) s_d[4 * ln.q + v][ln.j] = e[v] * gelu_d(z[0][v]);
      hidden_grad(s_a[0], s_e, ln, G + OFF_W2, G + OFF_B2, first);
    }
    __syncthreads();
    // first layer: dW1[k][j] = sum_s a0[s][k] dz1[s][j]
    {
      const int k1 = t >> 7, j = t & (H - 1);  // NT = NI H elements
      float g = 0.0f;
#pragma unroll
      for (int i = 0; i < TS; ++i) g = fmaf(s_a0[i][k1], s_d[i][j], g);
      gput(&G[OFF_W1 + t], g, first);
      if (k1 == 0) {
        float b = 0.0f;
#pragma unroll
        for (int i = 0; i < TS; ++i) b += s_d[i][j];
        gput(&G[OFF_B1 + j], b, first);
      }
    }
    __syncthreads();  // LDS reused by the next tile
  }
  // loss partial of this workgroup (wavefront 0 holds it)
  if (t < 64) {
    for (int off = 32; off > 0; off >>= 1) lacc += __shfl_down(lacc, off, 64);
    if (t == 0) lpart[blockIdx.x] = s_bad ? NAN : lacc;
  }
}
static_assert(NI == NO && TS * NI == 64, "wavefront 0 holds a tile's inputs and targets");
static_assert(NT == H * NO && NT == NI * H && NT == 4 * H, "element per thread phases");

__device__ __forceinline__ void adam_update(float* __restrict__ P, float* __restrict__ M,
                                            float* __restrict__ V, int p, float g, float lr,
                                            float b1, float b2, float eps, float bc1, float bc2) {
  const float m = b1 * M[p] + (1.0f - b1) * g;
  const float v = b2 * V[p] + (1.0f - b2) * g * g;
  M[p] = m;
  V[p] = v;
  P[p] -= lr * (m / bc1) / (sqrtf(v / bc2) + eps);
}

struct Adam {
  float *P, *M, *V;
  float lr, b1, b2, eps, bc1, bc2;
};

// Gradient from the slices, in their order; ADAM = 1: and the update of the
// parameters with it (a training step saves the launch and the gradient's
// round trip).
template <int ADAM>
__global__ void k_mlp_reduce(const float* __restrict__ part, const float* __restrict__ lpart,
                             int nblk, float scale, float* __restrict__ grad,
                             float* __restrict__ loss, const Adam ad) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p < NPARAM) {
    float g = 0.0f;
#pragma unroll 8
    for (int b = 0; b < nblk; ++b) g += part[(size_t)b * NPARAM + p];
    grad[p] = g;
    if constexpr (ADAM)
      adam_update(ad.P, ad.M, ad.V, p, g, ad.lr, ad.b1, ad.b2, ad.eps, ad.bc1, ad.bc2);
  }
  if (p == 0 && loss) {
    float s = 0.0f;
    for (int b = 0; b < nblk; ++b) s += lpart[b];
    *loss = s * scale;
  }
}

__global__ void k_mlp_adam(const float* __restrict__ G, const Adam ad) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p < NPARAM)
    adam_update(ad.P, ad.M, ad.V, p, G[p], ad.lr, ad.b1, ad.b2, ad.eps, ad.bc1, ad.bc2);
}

Norm to_norm(const lbm_mlp_norm* n) {
  Norm r;
  for (int i = 0; i < NI; ++i) {
    r.xs[i] = n->x_shift[i];
    r.xk[i] = n->x_scale[i];
  }
  for (int i = 0; i < NO; ++i) {
    r.ys[i] = n->y_shift[i];
    r.yk[i] = n->y_scale[i];
  }
  return r;
}

bool norm_ok(const lbm_mlp_norm* n) {
  for (int i = 0; i < NO; ++i)
    if (!(n->y_scale[i] != 0.0f) || !isfinite(n->y_scale[i]) || !isfinite(n->y_shift[i]))
      return false;
  for (int i = 0; i < NI; ++i)
    if (!isfinite(n->x_scale[i]) || !isfinite(n->x_shift[i])) return false;
  return true;
}

int grad_blocks(int n) {
  const int tiles = (n + TS - 1) / TS;
  return tiles < MAX_GRAD_BLOCKS ? tiles : MAX_GRAD_BLOCKS;
}

size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

// Workspace layout of a gradient over n samples: per-workgroup gradient
// slices, then the per-workgroup loss partials.
size_t part_bytes(int g) { return align256((size_t)g * NPARAM * sizeof(float)); }

lbm_status grad_args_ok(const float* d_params, const lbm_mlp_norm* norm, const float* d_x,
                        const float* d_y, int32_t n_rows, const int32_t* d_idx, int32_t n,
                        const float* d_grad, int32_t flags) {
  if (!d_params || !norm || !d_x || !d_y || !d_grad || n < 1 || n_rows < 1 ||
      (!d_idx && n > n_rows) || (flags & ~LBM_MLP_BF16))
    return LBM_ERR_INVALID_ARG;
  if (!norm_ok(norm)) return LBM_ERR_INVALID_ARG;
  return LBM_OK;
}

// The same with a caller workspace.
lbm_status grad_ws_ok(const float* d_params, const lbm_mlp_norm* norm, const float* d_x,
                      const float* d_y, int32_t n_rows, const int32_t* d_idx, int32_t n,
                      const float* d_grad, int32_t flags, const void* ws, size_t bytes) {
  const lbm_status s = grad_args_ok(d_params, norm, d_x, d_y, n_rows, d_idx, n, d_grad, flags);
  if (s != LBM_OK) return s;
  const int g = grad_blocks(n);
  const size_t need = part_bytes(g) + align256((size_t)g * sizeof(float));
  if (!ws || bytes < need || ((uintptr_t)ws % 256) != 0) return LBM_ERR_WORKSPACE;
  return LBM_OK;
}

Adam make_adam(float* d_params, float* d_m, float* d_v, int64_t t, float lr, float b1, float b2,
               float eps) {
  const float bc1 = (float)(1.0 - pow((double)b1, (double)t));
  const float bc2 = (float)(1.0 - pow((double)b2, (double)t));
  return Adam{d_params, d_m, d_v, lr, b1, b2, eps, bc1, bc2};
}

// The gradient kernels of lbm_mlp_grad on a scratch area `ws` laid out as
// above (arguments already checked), with the Adam update if one is given.
lbm_status grad_launch(const float* d_params, const lbm_mlp_norm* norm, const float* d_x,
                       const float* d_y, int32_t n_rows, const int32_t* d_idx, int32_t n,
                       float* d_grad, float* d_loss, int32_t flags, char* ws, hipStream_t st,
                       const Adam* adam = nullptr) {
  const Norm nm = to_norm(norm);
  const int g = grad_blocks(n);
  float* part = (float*)ws;
  float* lpart = (float*)(ws + part_bytes(g));
  const float scale = 1.0f / (4.0f * (float)n);
  if (flags & LBM_MLP_BF16)
    hipLaunchKernelGGL(k_mlp_grad<1>, dim3(g), dim3(NT), 0, st, d_params, nm, d_x, d_y, d_idx,
                       n, n_rows, scale, part, lpart);
  else
    hipLaunchKernelGGL(k_mlp_grad<0>, dim3(g), dim3(NT), 0, st, d_params, nm, d_x, d_y, d_idx,
                       n, n_rows, scale, part, lpart);
  const dim3 rg((NPARAM + 255) / 256), rb(256);
  if (adam)
    hipLaunchKernelGGL(k_mlp_reduce<1>, rg, rb, 0, st, part, lpart, g, scale, d_grad, d_loss, *adam);
  else
    hipLaunchKernelGGL(k_mlp_reduce<0>, rg, rb, 0, st, part, lpart, g, scale, d_grad, d_loss, Adam{});
  return hipGetLastError() == hipSuccess ? LBM_OK : LBM_ERR_HIP;
}

// ---- allocation-free gradient ----------------------------------------------
// lbm_mlp_grad_noalloc keeps the gradient partials in this file-scope device
// array instead of a caller workspace: room for the partials of
// LBM_MLP_NOALLOC_MAX_N samples (64 workgroup slices, about 8.4 MiB).  Every
// GPU the library runs on holds its own copy until the process ends.  In
// host code `scratch` is only a host-side stand-in for the symbol; kernels
// get its device address, looked up once per device below.
constexpr int NOALLOC_BLOCKS = (LBM_MLP_NOALLOC_MAX_N + TS - 1) / TS;
static_assert(NOALLOC_BLOCKS <= MAX_GRAD_BLOCKS, "no-alloc bound");
constexpr size_t NOALLOC_BYTES =
    ((size_t)NOALLOC_BLOCKS * NPARAM * sizeof(float) + 255) / 256 * 256 +
    ((size_t)NOALLOC_BLOCKS * sizeof(float) + 255) / 256 * 256;
static __device__ __align__(256) unsigned char scratch[NOALLOC_BYTES];

constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mu;
char* g_scratch_ptr[MAX_DEVICES] = {};

// Device address of `scratch` on device dev: hipGetSymbolAddress with dev
// current, on the first call for dev; later calls reuse the stored pointer.
lbm_status scratch_on(int dev, char** out) {
  if (dev < 0 || dev >= MAX_DEVICES) return LBM_ERR_UNSUPPORTED;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    int cur = -1;
    if (hipGetDevice(&cur) != hipSuccess) return LBM_ERR_HIP;
    if (cur != dev && hipSetDevice(dev) != hipSuccess) return LBM_ERR_HIP;
    void* ptr = nullptr;
    hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (cur != dev) (void)hipSetDevice(cur);
    if (e != hipSuccess || !ptr) return LBM_ERR_HIP;
    g_scratch_ptr[dev] = (char*)ptr;
  }
  *out = g_scratch_ptr[dev];
  return LBM_OK;
}

}  // namespace mlpk

using namespace mlpk;

extern "C" {

lbm_status lbm_mlp_workspace_bytes(int32_t n, size_t* bytes) {
  if (n < 1 || !bytes) return LBM_ERR_INVALID_ARG;
  const int g = grad_blocks(n);
  *bytes = align256((size_t)g * NPARAM * sizeof(float)) + align256((size_t)g * sizeof(float));
  return LBM_OK;
}

lbm_status lbm_mlp_forward(const float* d_params, const lbm_mlp_norm* norm, const float* d_x,
                           int32_t n, float* d_y, int32_t flags, void* hip_stream) {
  if (!d_params || !norm || n < 0 || (n > 0 && (!d_x || !d_y)) || (flags & ~LBM_MLP_BF16))
    return LBM_ERR_INVALID_ARG;
  if (!norm_ok(norm)) return LBM_ERR_INVALID_ARG;
  if (n == 0) return LBM_OK;
  hipStream_t st = (hipStream_t)hip_stream;
  const Norm nm = to_norm(norm);
  // each workgroup fetches 130 KB of weights: at most 512 of them walk the tiles
  const int tiles = (n + TS - 1) / TS, nb = tiles < 512 ? tiles : 512;
  if (flags & LBM_MLP_BF16)
    hipLaunchKernelGGL(k_mlp_forward<1>, dim3(nb), dim3(NT), 0, st, d_params, nm, d_x, n, d_y);
  else
    hipLaunchKernelGGL(k_mlp_forward<0>, dim3(nb), dim3(NT), 0, st, d_params, nm, d_x, n, d_y);
  return hipGetLastError() == hipSuccess ? LBM_OK : LBM_ERR_HIP;
}

lbm_status lbm_mlp_grad(const float* d_params, const lbm_mlp_norm* norm, const float* d_x,
                        const float* d_y, int32_t n_rows, const int32_t* d_idx, int32_t n,
                        float* d_grad, float* d_loss, int32_t flags, void* d_workspace,
                        size_t bytes, void* hip_stream) {
  const lbm_status s = grad_ws_ok(d_params, norm, d_x, d_y, n_rows, d_idx, n, d_grad, flags,
                                  d_workspace, bytes);
  if (s != LBM_OK) return s;
  return grad_launch(d_params, norm, d_x, d_y, n_rows, d_idx, n, d_grad, d_loss, flags,
                     (char*)d_workspace, (hipStream_t)hip_stream);
}

lbm_status lbm_mlp_grad_noalloc(const float* d_params, const lbm_mlp_norm* norm,
                                const float* d_x, const float* d_y, int32_t n_rows,
                                const int32_t* d_idx, int32_t n, float* d_grad, float* d_loss,
                                int32_t flags, void* hip_stream) {
  lbm_status s = grad_args_ok(d_params, norm, d_x, d_y, n_rows, d_idx, n, d_grad, flags);
  if (s != LBM_OK) return s;
  if (n > LBM_MLP_NOALLOC_MAX_N) return LBM_ERR_WORKSPACE;
  hipStream_t st = (hipStream_t)hip_stream;
  int dev = -1;
  if (st) {
    if (hipStreamGetDevice(st, &dev) != hipSuccess) return LBM_ERR_HIP;
  } else if (hipGetDevice(&dev) != hipSuccess) {
    return LBM_ERR_HIP;
  }
  char* ws = nullptr;
  if ((s = scratch_on(dev, &ws)) != LBM_OK) return s;
  return grad_launch(d_params, norm, d_x, d_y, n_rows, d_idx, n, d_grad, d_loss, flags, ws, st);
}

lbm_status lbm_mlp_adam(float* d_params, float* d_m, float* d_v, const float* d_grad, int64_t t,
                        float lr, float beta1, float beta2, float eps, void* hip_stream) {
  if (!d_params || !d_m || !d_v || !d_grad || t < 1 || !(lr >= 0.0f) || !(beta1 >= 0.0f) ||
      !(beta1 < 1.0f) || !(beta2 >= 0.0f) || !(beta2 < 1.0f) || !(eps > 0.0f))
    return LBM_ERR_INVALID_ARG;
  const Adam ad = make_adam(d_params, d_m, d_v, t, lr, beta1, beta2, eps);
  hipLaunchKernelGGL(k_mlp_adam, dim3((NPARAM + 255) / 256), dim3(256), 0,
                     (hipStream_t)hip_stream, d_grad, ad);
  return hipGetLastError() == hipSuccess ? LBM_OK : LBM_ERR_HIP;
}

lbm_status lbm_mlp_train_step(float* d_params, float* d_m, float* d_v, int64_t t, float lr,
                              const lbm_mlp_norm* norm, const float* d_x, const float* d_y,
                              int32_t n_rows, const int32_t* d_idx, int32_t n, float* d_grad,
                              float* d_loss, int32_t flags, void* d_workspace, size_t bytes,
                              void* hip_stream) {
  if (!d_m || !d_v || t < 1 || !(lr >= 0.0f)) return LBM_ERR_INVALID_ARG;
  lbm_status s = grad_ws_ok(d_params, norm, d_x, d_y, n_rows, d_idx, n, d_grad, flags, d_workspace,
                            bytes);
  if (s != LBM_OK) return s;
  const Adam ad = make_adam(d_params, d_m, d_v, t, lr, 0.9f, 0.999f, 1e-8f);
  return grad_launch(d_params, norm, d_x, d_y, n_rows, d_idx, n, d_grad, d_loss, flags,
                     (char*)d_workspace, (hipStream_t)hip_stream, &ad);
}

}  // extern "C"
