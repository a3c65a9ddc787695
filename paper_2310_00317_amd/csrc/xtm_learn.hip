// xtm_learn.hip -- gfx950 kernels of the learned early-stop path: early-turn
// features, the 16-128-128-1 loss predictor (BF16 MFMA operands, FP32
// accumulation) with its training step, and particle retirement.
//
// Rounding points of the network (shared with the reference): every GEMM
// operand (standardised inputs, activations, weights, back-propagated
// signals) is rounded FP32 -> BF16 to nearest even; products accumulate in
// FP32; bias, ReLU, sigmoid and loss are FP32.
//
// Matrix-core tiles: v_mfma_f32_16x16x16_bf16 with the operand layout
//   A (16 x 16, rows m, cols k): lane l holds A[l % 16][4 (l / 16) + j], j = 0..3
//   B (16 x 16, rows k, cols n): lane l holds B[4 (l / 16) + j][l % 16]
//   D (16 x 16):                 lane l holds D[4 (l / 16) + j][l % 16]
// so the D of a product is, element for element, the B operand of the next
// one, and the same registers taken as A are the transpose.  Every product
// below is written in the orientation whose D the next product reads as it
// lies: activations pass from layer to layer in registers.
#include <cmath>
#include <mutex>

#include "xtm_internal.h"
#include "xtm_maps.h"

namespace xtm {

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef short bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// parameter vector layout (FP32): W1[16][128], b1[128], W2[128][128], b2[128], w3[128], b3
constexpr int kIn = 16, kH = 128;
constexpr int oW1 = 0, oB1 = oW1 + kIn * kH, oW2 = oB1 + kH, oB2 = oW2 + kH * kH, oW3 = oB2 + kH,
              oB3 = oW3 + kH, kParams = oB3 + 1;
static_assert(kParams == 18817, "parameter count");
constexpr int kSamplesPerBlock = 64;  // rows of one partial gradient: 4 waves x 16
constexpr int kTiles = kH / 16;       // 16-neuron tiles of a hidden layer

__device__ __forceinline__ float bf16_value(float f) {  // rounded to bf16, as FP32
  return (float)(__bf16)f;
}
// Two values to a conversion (written value by value, the compiler converts
// each alone and merges the pairs with a permute: three operations for one).
__device__ __forceinline__ bf16x4 bf16_pack(float a, float b, float c, float d) {
  typedef float f2 __attribute__((ext_vector_type(2)));
  typedef __bf16 b2 __attribute__((ext_vector_type(2)));
  typedef unsigned int u2 __attribute__((ext_vector_type(2)));
  const u2 v = {__builtin_bit_cast(unsigned int, __builtin_convertvector((f2{a, b}), b2)),
                __builtin_bit_cast(unsigned int, __builtin_convertvector((f2{c, d}), b2))};
  return __builtin_bit_cast(bf16x4, v);
}
__device__ __forceinline__ bf16x8 bf16_join(bf16x4 lo, bf16x4 hi) {
  return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}
__device__ __forceinline__ float bf16_at(bf16x4 v, int j) {
  return __uint_as_float((unsigned int)(unsigned short)v[j] << 16);
}
__device__ __forceinline__ f32x4 mfma16(bf16x4 a, bf16x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

// The forward network in LDS, the weights as operand fragments (8 bytes per
// lane, 64 lanes of a fragment side by side: conflict-free reads; W2's in pairs,
// 16 bytes a read).  Lane l of a fragment holds four consecutive k of its column
// l % 16:
//   w1[nt][l]         W1[4 q + j][16 nt + l % 16]            (q = l / 16)
//   w2[nt][kt / 2][l] W2[16 kt + 4 q + j][16 nt + l % 16], kt even low, odd high
struct NetLds {
  bf16x4 w1[kTiles][64];
  bf16x8 w2[kTiles][kTiles / 2][64];
  float b1[kH], b2[kH], w3[kH];  // w3 already rounded to bf16 values
  float b3;
};

__device__ __forceinline__ float4 load4(const float* p) {
  return make_float4(p[0], p[1], p[2], p[3]);
}

__device__ void load_net(NetLds& s, const float* __restrict__ th) {
  // group g: four rows of one column (neighbouring threads neighbouring columns)
  for (int g = threadIdx.x; g < kIn / 4 * kH; g += blockDim.x) {
    const int q = g / kH, n = g % kH;
    const float* w = th + oW1 + 4 * q * kH + n;
    s.w1[n / 16][q * 16 + n % 16] = bf16_pack(w[0], w[kH], w[2 * kH], w[3 * kH]);
  }
  // eight rows of four columns at a time, a thread's sixteen 16-byte reads all in
  // flight (256 threads)
  float4 v[2][8];
#pragma unroll
  for (int m = 0; m < 2; ++m) {
    const int g = (int)threadIdx.x + 256 * m, k8 = g / (kH / 4), n = 4 * (g % (kH / 4));
    const int k = 32 * (k8 / 4) + 4 * (k8 % 4);  // rows k .. k + 3 and k + 16 .. k + 19
#pragma unroll
    for (int j = 0; j < 8; ++j) v[m][j] = load4(th + oW2 + (k + j % 4 + 16 * (j / 4)) * kH + n);
  }
#pragma unroll
  for (int m = 0; m < 2; ++m) {
    const int g = (int)threadIdx.x + 256 * m, k8 = g / (kH / 4), n = 4 * (g % (kH / 4));
    bf16x8* to = &s.w2[n / 16][k8 / 4][(k8 % 4) * 16 + n % 16];
    const float4* r = v[m];
    to[0] = bf16_join(bf16_pack(r[0].x, r[1].x, r[2].x, r[3].x),
                      bf16_pack(r[4].x, r[5].x, r[6].x, r[7].x));
    to[1] = bf16_join(bf16_pack(r[0].y, r[1].y, r[2].y, r[3].y),
                      bf16_pack(r[4].y, r[5].y, r[6].y, r[7].y));
    to[2] = bf16_join(bf16_pack(r[0].z, r[1].z, r[2].z, r[3].z),
                      bf16_pack(r[4].z, r[5].z, r[6].z, r[7].z));
    to[3] = bf16_join(bf16_pack(r[0].w, r[1].w, r[2].w, r[3].w),
                      bf16_pack(r[4].w, r[5].w, r[6].w, r[7].w));
  }
  for (int i = threadIdx.x; i < kH; i += blockDim.x) {
    s.b1[i] = th[oB1 + i];
    s.b2[i] = th[oB2 + i];
    s.w3[i] = bf16_value(th[oW3 + i]);
  }
  if (threadIdx.x == 0) s.b3 = th[oB3];
}

// What lanes of a wave wrote to LDS is there for its other lanes from here on (a
// wave's LDS operations run in order: no instruction, but the compiler is told).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ float relu(float z) { return z > 0.f ? z : 0.f; }

// Features 4 q .. 4 q + 3 of row `row`; the first row's when `on` is false (a
// read every lane can do, so the rows' reads need no branches).
__device__ __forceinline__ float4 read_x(const float* __restrict__ X, int64_t row, bool on, int q) {
  return load4(X + (on ? row : 0) * kIn + 4 * q);
}

// Standardised inputs (of zeros when `on` is false): the operand of one lane.
__device__ __forceinline__ bf16x4 standard_x(const float4& x, bool on, const float4& mean,
                                             const float4& inv) {
  const float x0 = on ? x.x : 0.f, x1 = on ? x.y : 0.f, x2 = on ? x.z : 0.f, x3 = on ? x.w : 0.f;
  return bf16_pack((x0 - mean.x) * inv.x, (x1 - mean.y) * inv.y, (x2 - mean.z) * inv.z,
                   (x3 - mean.w) * inv.w);
}

// Activations of four neurons (16 nt + 4 q ..) of one sample: bias, ReLU, bf16.
__device__ __forceinline__ bf16x4 activate(const f32x4& c, const float* bias) {
  return bf16_pack(relu(c[0] + bias[0]), relu(c[1] + bias[1]), relu(c[2] + bias[2]),
                   relu(c[3] + bias[3]));
}

// Forward pass, T tiles of 16 rows per wave: both layers as weights^T times
// activations^T, so a layer's D (neurons down, samples across) is the next
// layer's B operand.  Each block loads the network once and then runs tiles
// blockIdx.x, blockIdx.x + gridDim.x, ...  T = 4 shares each fragment read among
// four products.
//   What bounds it: 72 matrix instructions a tile, 31 us for 2^20 rows at their
// rate, and about as long in vector instructions (bias, ReLU, rounding, output
// layer).  A layer-2 tile is therefore activated while the next one's products
// run (three vector instructions to a product); the products go to vector
// registers (with room for one wave a SIMD, the compiler takes accumulation
// registers and copies every value out); the rows come a pass ahead.
//   us for 2^20 rows: 757 when every operand was staged element by element
// through LDS; 83 with the fragments; 63 with conversions and fragments in pairs,
// the products in vector registers and the rows ahead; 54, 0.71 PFLOP/s, with
// the activation between the products.  Two tiles a wave and twice the waves do
// not replace that: 57.  The 32-deep product would give 12 us less, but adds in
// another order, and some hidden values then round the other way.
//   __launch_bounds__: two waves a SIMD.
template <int T>
__global__ void __launch_bounds__(256, 2) k_mlp_forward(const float* __restrict__ theta,
                                                     const float* __restrict__ norm,
                                                     const float* __restrict__ X, int64_t B,
                                                     float* __restrict__ logit) {
  __shared__ NetLds net;
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  const int col = l & 15, q = l >> 4;
  const float4 mean = load4(norm + 4 * q), inv = load4(norm + kIn + 4 * q);
  const int64_t per_block = 64 * T, step = gridDim.x * per_block;
  int64_t s0 = blockIdx.x * per_block + w * 16 * T + col;  // this lane's first sample
  float4 in[T];
#pragma unroll
  for (int t = 0; t < T; ++t) in[t] = read_x(X, s0 + 16 * t, s0 + 16 * t < B, q);
  load_net(net, theta);
  __syncthreads();
  for (int64_t base = blockIdx.x * per_block; base < B; base += step, s0 += step) {
    bf16x4 x[T], h[T][kTiles];
#pragma unroll
    for (int t = 0; t < T; ++t) x[t] = standard_x(in[t], s0 + 16 * t < B, mean, inv);
    if (base + step < B) {  // the next pass's rows, under this one's products
#pragma unroll
      for (int t = 0; t < T; ++t)
        in[t] = read_x(X, s0 + step + 16 * t, s0 + step + 16 * t < B, q);
    }
#pragma unroll
    for (int nt = 0; nt < kTiles; ++nt) {
      const bf16x4 a = net.w1[nt][l];
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const f32x4 c = mfma16(a, x[t], f32x4{0.f, 0.f, 0.f, 0.f});
        h[t][nt] = activate(c, net.b1 + 16 * nt + 4 * q);
      }
    }
    float z[T];
#pragma unroll
    for (int t = 0; t < T; ++t) z[t] = 0.f;
    f32x4 p[T];  // the tile before, activated between this one's products
    const auto finish = [&](int nt) {
      const float* w3 = net.w3 + 16 * nt + 4 * q;
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const bf16x4 v = activate(p[t], net.b2 + 16 * nt + 4 * q);
#pragma unroll
        for (int j = 0; j < 4; ++j) z[t] += bf16_at(v, j) * w3[j];
      }
    };
    const auto products = [&](int nt, f32x4* c) {
#pragma unroll
      for (int t = 0; t < T; ++t) c[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kt = 0; kt < kTiles; kt += 2) {
        const bf16x8 a = net.w2[nt][kt / 2][l];
#pragma unroll
        for (int t = 0; t < T; ++t) c[t] = mfma16(a.lo, h[t][kt], c[t]);
#pragma unroll
        for (int t = 0; t < T; ++t) c[t] = mfma16(a.hi, h[t][kt + 1], c[t]);
      }
    };
    products(0, p);
#pragma unroll 1
    for (int nt = 1; nt < kTiles; ++nt) {
      f32x4 c[T];
      products(nt, c);
      finish(nt - 1);
#pragma unroll
      for (int t = 0; t < T; ++t) p[t] = c[t];
#pragma unroll
      for (int i = 0; i < kTiles * T; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);  // a product
        __builtin_amdgcn_sched_group_barrier(0x2, 3, 0);  // three vector operations
      }
    }
    finish(kTiles - 1);
#pragma unroll
    for (int t = 0; t < T; ++t) {
      float v = z[t];
      v += __shfl_xor(v, 16, 64);
      v += __shfl_xor(v, 32, 64);
      if (q == 0 && s0 + 16 * t < B) logit[s0 + 16 * t] = v + net.b3;
    }
  }
}

// Training step of 64 rows per block, 16 per wave, split over gridDim.y blocks
// that each hold `kTiles / gridDim.y` of the 16-wide column tiles of the weight
// gradients (every one of them runs the forward pass; a batch of a few
// thousand rows has fewer 64-row blocks than the chip has CUs).  Operands:
//   H1^T, H2^T  (D of weights^T x activations^T): B operand of the next layer
//   H1, dZ2, dZ1 (D of the same registers as A): rows are samples, so they are
//                operands of the products that contract over samples:
//                gW2 = H1^T dZ2, gW1 = X^T dZ1
// H1 and dZ2 of the four waves meet in LDS for gW2's contraction over the
// block's 64 rows.  What bounds it: latency, a block's chain from the weights
// (75 KB) over three small products to its share of the partial gradient;
// 81 us a call of 4,096 rows (16,384: 141) in the form that staged every
// element through LDS, now 20 (16,384: 38), its reduction included.  Every sum
// keeps that form's order, so a training run gives the same bits (with the
// logit's sum in another order, 3 % faster, the rounding of some activation
// fell the other way after some tens of steps, and the weights went apart).
struct GradLds {
  NetLds net;
  bf16x4 w2r[kTiles][kTiles][64];   // W2[16 mt + l % 16][16 kt + 4 q + j], own tiles mt
  bf16x4 h1[4][kTiles][64];         // per wave: H1[4 q + j][16 mt + l % 16]
  bf16x4 dz2[4][kTiles][64];        // per wave: dZ2[4 q + j][16 nt + l % 16], own tiles nt
  bf16x4 dz1[4][kTiles][64];        // per wave: dZ1, own tiles
  unsigned short x[4][16][kIn + 4]; // per wave: rows of X (bf16)
  unsigned short h2[kSamplesPerBlock][kH + 8];  // rows of H2 (bf16)
  float gb1[4][kH];                 // per-wave column sums
  float dz3[4][16], lossv[4][16];
};

// Per-block partial gradient (mean over the whole batch B) into part[blockIdx.x][kParams]
// and the block's summed loss into loss_part[blockIdx.x].  perm: row r of the
// batch is row perm[r] of (X, Y); null: row r.
__global__ void __launch_bounds__(256) k_mlp_grad(const float* __restrict__ theta,
                                                  const float* __restrict__ norm,
                                                  const float* __restrict__ X,
                                                  const float* __restrict__ Y,
                                                  const int32_t* __restrict__ perm, int64_t B,
                                                  float pos_weight, float* __restrict__ part,
                                                  float* __restrict__ loss_part) {
  __shared__ GradLds s;
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  const int col = l & 15, q = l >> 4;
  const int own = kTiles / (int)gridDim.y, t0 = (int)blockIdx.y * own;  // own tiles t0 .. t0 + own
  // the rows first: a row's place and then its words are two latencies, under
  // the weights' one
  const int64_t row = (int64_t)blockIdx.x * kSamplesPerBlock + 16 * w + col;  // this lane's sample
  const bool on = row < B;
  const int64_t src = on ? (perm ? perm[row] : row) : 0;
  const float4 mean = load4(norm + 4 * q), inv = load4(norm + kIn + 4 * q);
  const bf16x4 x = standard_x(read_x(X, src, on, q), on, mean, inv);
  const float y = on ? Y[src] : 0.f;
  load_net(s.net, theta);
  for (int g = threadIdx.x; g < own * 16 * (kH / 4); g += blockDim.x) {
    const int r = t0 * 16 + g / (kH / 4), c4 = g % (kH / 4);
    const float4 v = load4(theta + oW2 + r * kH + 4 * c4);
    s.w2r[r / 16][c4 / 4][(c4 % 4) * 16 + r % 16] = bf16_pack(v.x, v.y, v.z, v.w);
  }
  *reinterpret_cast<bf16x4*>(&s.x[w][col][4 * q]) = x;
  __syncthreads();
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  bf16x4 h1t[kTiles];
#pragma unroll
  for (int nt = 0; nt < kTiles; ++nt) {
    const bf16x4 a = s.net.w1[nt][l];
    h1t[nt] = activate(mfma16(a, x, zero), s.net.b1 + 16 * nt + 4 * q);
    const f32x4 c = mfma16(x, a, zero);  // samples down, neurons across
    const float b = s.net.b1[16 * nt + col];
    s.h1[w][nt][l] =
        bf16_pack(relu(c[0] + b), relu(c[1] + b), relu(c[2] + b), relu(c[3] + b));
  }
  bf16x4 h2t[kTiles];
#pragma unroll
  for (int nt = 0; nt < kTiles; ++nt) {
    f32x4 c = zero;
#pragma unroll
    for (int kt = 0; kt < kTiles; kt += 2) {
      const bf16x8 a = s.net.w2[nt][kt / 2][l];
      c = mfma16(a.hi, h1t[kt + 1], mfma16(a.lo, h1t[kt], c));
    }
    h2t[nt] = activate(c, s.net.b2 + 16 * nt + 4 * q);
    *reinterpret_cast<bf16x4*>(&s.h2[16 * w + col][16 * nt + 4 * q]) = h2t[nt];
  }
  // the logit of this lane's sample, the neurons in order (training amplifies
  // a rounding that falls the other way, so every sum of the step has one order):
  // its row comes from four lanes of this wave
  wave_sync();
  float z = 0.f;
#pragma unroll
  for (int k = 0; k < kH; k += 4) {
    const bf16x4 h = *reinterpret_cast<const bf16x4*>(&s.h2[16 * w + col][k]);
#pragma unroll
    for (int j = 0; j < 4; ++j) z += bf16_at(h, j) * s.net.w3[k + j];
  }
  z += s.net.b3;
  // dL/dz3 of this lane's sample (the four quads hold the same)
  float d = 0.f, lv = 0.f;
  if (on) {
    const float sg = 1.0f / (1.0f + expf(-z));
    d = (sg * (pos_weight * y + (1.0f - y)) - pos_weight * y) / (float)B;
    const float lz = log1pf(expf(-fabsf(z)));
    const float sp_neg = fmaxf(-z, 0.f) + lz, sp_pos = fmaxf(z, 0.f) + lz;
    lv = pos_weight * y * sp_neg + (1.0f - y) * sp_pos;
  }
  if (q == 0) {
    s.dz3[w][col] = d;
    s.lossv[w][col] = lv;
  }
  __syncthreads();
  const float dq = bf16_value(d);  // this lane's sample across
  float dqr[4];                    // the four samples down
#pragma unroll
  for (int j = 0; j < 4; ++j) dqr[j] = bf16_value(s.dz3[w][4 * q + j]);
  // dZ2 transposed: the operand of dH1 = dZ2 W2^T
  bf16x4 dz2t[kTiles];
#pragma unroll
  for (int nt = 0; nt < kTiles; ++nt) {
    const float* w3 = s.net.w3 + 16 * nt + 4 * q;
    float v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = bf16_at(h2t[nt], j) > 0.f ? dq * w3[j] : 0.f;
    dz2t[nt] = bf16_pack(v[0], v[1], v[2], v[3]);
  }
  // own tiles, samples down: dZ2, and dZ1 with b1's sums
  for (int nt = t0; nt < t0 + own; ++nt) {
    const int n = 16 * nt + col;
    const float w3 = s.net.w3[n];
    float v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = s.h2[16 * w + 4 * q + j][n] ? dqr[j] * w3 : 0.f;
    s.dz2[w][nt][l] = bf16_pack(v[0], v[1], v[2], v[3]);
    f32x4 g = zero;
#pragma unroll
    for (int kt = 0; kt < kTiles; ++kt) g = mfma16(dz2t[kt], s.w2r[nt][kt][l], g);
    const bf16x4 h1 = s.h1[w][nt][l];
    float gb1 = 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      v[j] = bf16_at(h1, j) > 0.f ? g[j] : 0.f;
      gb1 += v[j];
    }
    s.dz1[w][nt][l] = bf16_pack(v[0], v[1], v[2], v[3]);
    gb1 += __shfl_xor(gb1, 16, 64);
    gb1 += __shfl_xor(gb1, 32, 64);
    if (q == 0) s.gb1[w][n] = gb1;
  }
  __syncthreads();
  float* g = part + (size_t)blockIdx.x * kParams;
  for (int n = 16 * t0 + (int)threadIdx.x; n < 16 * (t0 + own); n += blockDim.x)
    g[oB1 + n] = ((s.gb1[0][n] + s.gb1[1][n]) + s.gb1[2][n]) + s.gb1[3][n];
  // own columns' b2 and w3 sums, the block's b3 and loss: rows in order
  const int cols = 16 * own;
  if ((int)threadIdx.x < 2 * cols) {
    const bool for_w3 = (int)threadIdx.x >= cols;
    const int n = 16 * t0 + (for_w3 ? (int)threadIdx.x - cols : (int)threadIdx.x);
    const float w3 = s.net.w3[n];
    float acc = 0.f;
#pragma unroll 16
    for (int r = 0; r < kSamplesPerBlock; ++r) {
      const float dr = bf16_value(s.dz3[r / 16][r % 16]);
      const unsigned short h = s.h2[r][n];
      const float hw = __uint_as_float((unsigned int)h << 16) * dr, hb = h ? dr * w3 : 0.f;
      acc += for_w3 ? hw : hb;
    }
    g[(for_w3 ? oW3 : oB2) + n] = acc;
  }
  if (blockIdx.y == 0 && (threadIdx.x == 191 || threadIdx.x == 255)) {
    const bool for_loss = threadIdx.x == 255;
    const float* v = for_loss ? &s.lossv[0][0] : &s.dz3[0][0];
    float acc = 0.f;
#pragma unroll 16
    for (int r = 0; r < kSamplesPerBlock; ++r) acc += v[r];
    if (for_loss) loss_part[blockIdx.x] = acc;
    else g[oB3] = acc;
  }
  // W2[j1][n2] = sum_s H1[s][j1] dZ2[s][n2], own n2 tiles, in steps of 16 rows
  for (int t = w; t < kTiles * own; t += 4) {
    const int mt = t % kTiles, nt = t0 + t / kTiles;
    f32x4 c = zero;
#pragma unroll
    for (int kt = 0; kt < 4; ++kt) c = mfma16(s.h1[kt][mt][l], s.dz2[kt][nt][l], c);
#pragma unroll
    for (int j = 0; j < 4; ++j) g[oW2 + (mt * 16 + 4 * q + j) * kH + nt * 16 + col] = c[j];
  }
  // W1[f][j1] = sum_s X[s][f] dZ1[s][j1], own j1 tiles
  for (int nt = t0 + w; nt < t0 + own; nt += 4) {
    f32x4 c = zero;
#pragma unroll
    for (int kt = 0; kt < 4; ++kt) {
      bf16x4 a;
#pragma unroll
      for (int j = 0; j < 4; ++j) a[j] = (short)s.x[kt][4 * q + j][col];
      c = mfma16(a, s.dz1[kt][nt][l], c);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) g[oW1 + (4 * q + j) * kH + nt * 16 + col] = c[j];
  }
}

// Sum over blocks b = 0..nb-1 (in order) of part[b][i]: the loads of 32
// partials in flight at a time (the sums of one parameter are one chain).
__device__ __forceinline__ float sum_parts(const float* __restrict__ part, int nb, size_t stride,
                                           int i) {
  float acc = 0.f;
  int b = 0;
  for (; b + 32 <= nb; b += 32) {
    float v[32];
#pragma unroll
    for (int k = 0; k < 32; ++k) v[k] = part[(size_t)(b + k) * stride + i];
#pragma unroll
    for (int k = 0; k < 32; ++k) acc += v[k];
  }
  for (; b < nb; ++b) acc += part[(size_t)b * stride + i];
  return acc;
}

__global__ void __launch_bounds__(64) k_mlp_reduce(const float* __restrict__ part, int nb,
                                                   const float* __restrict__ loss_part,
                                                   float* __restrict__ grad,
                                                   float* __restrict__ loss, int64_t B) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < kParams) grad[i] = sum_parts(part, nb, kParams, i);
  if (i == kParams && loss) *loss = sum_parts(loss_part, nb, 1, 0) / (float)B;
}

// Adam (Kingma & Ba): m <- b1 m + (1-b1) g, v <- b2 v + (1-b2) g^2,
// theta <- theta - lr mhat / (sqrt(vhat) + eps), bias-corrected with step t >= 1
// (c.x = 1 - b1^t, c.y = 1 - b2^t; a training epoch's from one launch).  The update is evaluated in
// FP64 from the FP32 masters and moments (b1 = 0.9, b2 = 0.999 exactly, not
// their FP32 roundings) and stored back in FP32.
constexpr double kB1 = 0.9, kB2 = 0.999, kEps = 1e-8;

__device__ __forceinline__ double2 adam_bias(int step) {
  return make_double2(1.0 - pow(kB1, (double)step), 1.0 - pow(kB2, (double)step));
}

__global__ void __launch_bounds__(256) k_adam_bias(double2* __restrict__ c, int first, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) c[i] = adam_bias(first + i);
}

__device__ __forceinline__ void adam_update(float* __restrict__ theta, float* __restrict__ m,
                                            float* __restrict__ v, int i, double g,
                                            const double2& c, float lr) {
  const double mi = kB1 * (double)m[i] + (1.0 - kB1) * g;
  const double vi = kB2 * (double)v[i] + (1.0 - kB2) * g * g;
  m[i] = (float)mi;
  v[i] = (float)vi;
  const double mh = mi / c.x;
  const double vh = vi / c.y;
  theta[i] = (float)((double)theta[i] - (double)lr * mh / (sqrt(vh) + kEps));
}

__global__ void __launch_bounds__(64) k_adam(float* __restrict__ theta, float* __restrict__ m,
                                             float* __restrict__ v,
                                             const float* __restrict__ grad, int step,
                                             float lr) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < kParams) adam_update(theta, m, v, i, grad[i], adam_bias(step), lr);
}

// The reduction of a training step and its update in one launch (the training
// loop keeps no gradient).
__global__ void __launch_bounds__(64) k_mlp_reduce_adam(const float* __restrict__ part, int nb,
                                                        const float* __restrict__ loss_part,
                                                        float* __restrict__ loss, int64_t B,
                                                        float* __restrict__ theta,
                                                        float* __restrict__ m,
                                                        float* __restrict__ v,
                                                        const double2* __restrict__ bias,
                                                        float lr) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < kParams) adam_update(theta, m, v, i, sum_parts(part, nb, kParams, i), *bias, lr);
  if (i == kParams && loss) *loss = sum_parts(loss_part, nb, 1, 0) / (float)B;
}

// He-normal initialisation: weights std sqrt(2/fan_in) times the Philox
// deviate of (seed, index j, 0, 0, 0); biases zero.
__global__ void __launch_bounds__(256) k_mlp_init(float* __restrict__ theta,
                                                  unsigned long long seed) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= kParams) return;
  double std = 0.0;
  if (i < oB1) std = sqrt(2.0 / kIn);
  else if (i >= oW2 && i < oB2) std = sqrt(2.0 / kH);
  else if (i >= oW3 && i < oB3) std = sqrt(2.0 / kH);
  theta[i] = std == 0.0 ? 0.0f : (float)(std * xtmm::gauss_at(seed, i, 0, 0, 0));
}

// ------------------------------------------------------------- features
constexpr int kWin = 512, kRecTurns = 1024;

// Three stages (half = stride, 2 stride, 4 stride) of the radix-2
// decimation-in-time transform on eight elements `stride` apart, the first of
// them at position `pos` of its group of `stride`: v0 +- w v1 with
// w = exp(-i 2 pi k / 512) = (cos, -sin) from tw.
template <int kStride>
__device__ __forceinline__ void fft_stages(float2 (&v)[8], int pos, const float2* tw) {
#pragma unroll
  for (int st = 0; st < 3; ++st) {
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      if (k & (1 << st)) continue;
      const int low = k & ((1 << st) - 1);
      const float2 w = tw[(pos + kStride * low) * (256 / (kStride << st))];
      const float2 v0 = v[k], v1 = v[k | (1 << st)];
      const float tr = w.x * v1.x + w.y * v1.y;
      const float ti = w.x * v1.y - w.y * v1.x;
      v[k | (1 << st)] = make_float2(v0.x - tr, v0.y - ti);
      v[k] = make_float2(v0.x + tr, v0.y + ti);
    }
  }
}

// G particles per workgroup of T threads: thread % G is the particle, and T / G
// threads share its turns.
constexpr int kStats = 10;
template <int G, int T>
struct FeatLds {
  float2 z[kWin][G];  // one transform of each particle
  float2 tw[kWin / 2];
  float win[kWin];
  double red[T / 64][kStats][G];
  float best[T / 64][G];
  int at[T / 64][G];
};

template <int G>
__device__ __forceinline__ double lanes_sum(double v) {
#pragma unroll
  for (int o = G; o < 64; o <<= 1) v += __shfl_xor(v, o, 64);
  return v;
}
template <int G>
__device__ __forceinline__ double lanes_max(double v) {
#pragma unroll
  for (int o = G; o < 64; o <<= 1) v = fmax(v, __shfl_xor(v, o, 64));
  return v;
}

// Second and third pass over the transform in s.z, then the peak bin (first
// index on ties) and Hann's three-point interpolation: ((k + d) / 512) mod 1
// for the threads below G.
template <int G, int T>
__device__ float tune_of(FeatLds<G, T>& s) {
  constexpr int kThreads = T / G;
  const int p = threadIdx.x % G;
  // (hidden from the optimiser, which would otherwise keep the twiddles of
  // every pass in registers from one transform to the next)
  int tl = threadIdx.x / G;
  asm volatile("" : "+v"(tl));
#pragma unroll
  for (int i = tl; i < kWin / 8; i += kThreads) {
    float2 v[8];
    const int base = (i / 8) * 64 + i % 8;
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = s.z[base + 8 * j][p];
    fft_stages<8>(v, i % 8, s.tw);
#pragma unroll
    for (int j = 0; j < 8; ++j) s.z[base + 8 * j][p] = v[j];
  }
  __syncthreads();
  float best = -1.f;
  int at = 0;
#pragma unroll
  for (int i = tl; i < kWin / 8; i += kThreads) {
    float2 v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = s.z[i + 64 * j][p];
    fft_stages<64>(v, i, s.tw);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int k = i + 64 * j;
      const float m = sqrtf(v[j].x * v[j].x + v[j].y * v[j].y);
      s.z[k][p].x = m;
      if (m > best || (m == best && k < at)) {
        best = m;
        at = k;
      }
    }
  }
#pragma unroll
  for (int o = G; o < 64; o <<= 1) {
    const float ob = __shfl_xor(best, o, 64);
    const int oa = __shfl_xor(at, o, 64);
    if (ob > best || (ob == best && oa < at)) {
      best = ob;
      at = oa;
    }
  }
  if ((threadIdx.x & 63) < G) {
    s.best[threadIdx.x >> 6][p] = best;
    s.at[threadIdx.x >> 6][p] = at;
  }
  __syncthreads();
  float q = 0.f;
  if (threadIdx.x < G) {
    for (int w = 1; w < T / 64; ++w) {
      const float ob = s.best[w][p];
      const int oa = s.at[w][p];
      if (ob > best || (ob == best && oa < at)) {
        best = ob;
        at = oa;
      }
    }
    const float am = s.z[(at + kWin - 1) % kWin][p].x, b = s.z[at][p].x,
                c = s.z[(at + 1) % kWin][p].x;
    const float d = 2.0f * (c - am) / (am + 2.0f * b + c);
    q = ((float)at + d) / (float)kWin;
    q = q - floorf(q);
  }
  __syncthreads();
  return q;
}

// Record [1024][4][n] (x, px, y, py at element 0 at the start of each turn)
// -> 16 features (definitions in include/xtm.h).  The action statistics are
// taken in FP64 from the FP32 record (sums of the differences from the first
// turn's action: one pass, no cancellation); the spectra are FP32 FFTs.
// tw[k] = (cos, sin)(2 pi k / 512) for k < 256, win[n] = sin^2(pi n / 512).
//   What bounds it: the record is read once, 16 KB per particle; a turn of one
// particle is 4 bytes in a row of n, so G = 8 neighbours share each 32-byte
// piece, and groups of neighbours are numbered within an XCD (blocks go round
// the eight XCDs), whose L2 then holds the rest of each 128-byte line.
// One particle per workgroup fetched every piece eight times over: 1,040 us
// for 20,000 particles, 0.32 TB/s; now 195 us, 1.7 TB/s, the rest of the
// time being the FP64 actions and the transforms between the barriers.  Eight
// butterflies' elements stay in registers for three stages, so a transform
// crosses LDS three times, not nine (same operations in the same order).
// Off: the type of a lane's offset within 64 turns (32 bits while 64 rows of
// 4 n floats stay below 4 GiB).
template <int G, int T, typename Off>
__global__ void __launch_bounds__(T, 4) k_features(const float* __restrict__ rec, int64_t n,
                                                  double bx, double ax, double by, double ay,
                                                  double emit, double r_ap,
                                                  const float2* __restrict__ tw,
                                                  const float* __restrict__ win,
                                                  float* __restrict__ out) {
  __shared__ FeatLds<G, T> s;
  constexpr int kThreads = T / G, kBlk = 64 / kThreads;
  const int64_t groups = (n + G - 1) / G, per_xcd = (groups + 7) / 8;
  const int64_t grp = (int64_t)(blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (grp >= groups) return;
  const int p = threadIdx.x % G, tl = threadIdx.x / G;
  const int64_t i = grp * G + p;
  const bool on = i < n;
  const int64_t ip = on ? i : n - 1;
  const float* __restrict__ r = rec + ip;
  for (int k = threadIdx.x; k < kWin / 2; k += T) s.tw[k] = tw[k];
  for (int k = threadIdx.x; k < kWin; k += T) s.win[k] = win[k];
  // normalised coordinates u = x / sqrt(b), pu = (a x + b px) / sqrt(b) and the
  // action (u^2 + pu^2) / 2, as (x^2 + (a x + b px)^2) / 2 b: products with the
  // reciprocals instead of four quotients a turn (202 us -> 195 us)
  const double rsx = 1.0 / sqrt(bx), rsy = 1.0 / sqrt(by), hbx = 0.5 / bx, hby = 0.5 / by;
  auto action = [](double x, double px, double a, double b, double rs, double hb, double& u,
                   double& pu) {
    const double l = fma(b, px, a * x);
    u = x * rs;
    pu = l * rs;
    return fma(l, l, x * x) * hb;
  };
  double u, pu;
  const double jx0 = action(r[0], r[n], ax, bx, rsx, hbx, u, pu);
  const double jy0 = action(r[2 * n], r[3 * n], ay, by, rsy, hby, u, pu);
  // sums of j - j0 and its square, the first and last quarter's j; maxima
  double d1x = 0.0, d2x = 0.0, f0x = 0.0, f1x = 0.0, d1y = 0.0, d2y = 0.0, f0y = 0.0, f1y = 0.0;
  double r2max = 0.0, amax = 0.0;
  float q[4];
  __syncthreads();
#pragma unroll 1
  for (int h = 0; h < 2; ++h) {
    float2 zy[kBlk][8];
    // sums of this half's first and second quarter
    double lx = 0.0, ly = 0.0, hx = 0.0, hy = 0.0;
#pragma unroll
    for (int b = 0; b < kBlk; ++b) {
      // elements 8 blk .. 8 blk + 7 of the bit-reversed order: turns 64 apart
      const int blk = tl + kThreads * b;
      const int tb = (int)(__brev((unsigned)blk) >> 26);
      float2 zx[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int rk = ((k & 1) << 2) | (k & 2) | (k >> 2), t = tb + 64 * rk;
        // a row common to the workgroup, and the lane's offset from it
        const float* __restrict__ row = rec + (size_t)(h * kWin + 64 * rk) * 4 * n;
        const Off at = (Off)tb * 4 * (Off)n + (Off)ip;
        const double x = row[at], px = row[n + at], y = row[2 * n + at], py = row[3 * n + at];
        double ux, pux, uy, puy;
        const double jx = action(x, px, ax, bx, rsx, hbx, ux, pux);
        const double jy = action(y, py, ay, by, rsy, hby, uy, puy);
        const double dx = jx - jx0, dy = jy - jy0;
        d1x += dx;
        d2x = fma(dx, dx, d2x);
        d1y += dy;
        d2y = fma(dy, dy, d2y);
        (rk < 4 ? lx : hx) += jx;
        (rk < 4 ? ly : hy) += jy;
        r2max = fmax(r2max, x * x + y * y);
        amax = fmax(amax, jx + jy);
        const float wv = s.win[t];
        zx[k] = make_float2(wv * (float)ux, -wv * (float)pux);
        zy[b][k] = make_float2(wv * (float)uy, -wv * (float)puy);
        // the sums are taken turn by turn (an empty constraint: the compiler
        // otherwise keeps every turn's actions in registers to sum them later)
        asm volatile("" : "+v"(d1x), "+v"(d2x), "+v"(d1y), "+v"(d2y), "+v"(lx), "+v"(ly),
                          "+v"(hx), "+v"(hy), "+v"(r2max), "+v"(amax));
      }
      fft_stages<1>(zx, 0, s.tw);
      fft_stages<1>(zy[b], 0, s.tw);
#pragma unroll
      for (int k = 0; k < 8; ++k) s.z[8 * blk + k][p] = zx[k];
    }
    if (h == 0) {
      f0x = lx;
      f0y = ly;
    } else {
      f1x = hx;
      f1y = hy;
    }
    __syncthreads();
    q[2 * h] = tune_of<G, T>(s);
#pragma unroll
    for (int b = 0; b < kBlk; ++b)
#pragma unroll
      for (int k = 0; k < 8; ++k) s.z[8 * (tl + kThreads * b) + k][p] = zy[b][k];
    __syncthreads();
    q[2 * h + 1] = tune_of<G, T>(s);
  }
  double v[kStats] = {d1x, d2x, f0x, f1x, d1y, d2y, f0y, f1y, r2max, amax};
#pragma unroll
  for (int k = 0; k < kStats; ++k) {
    v[k] = k < 8 ? lanes_sum<G>(v[k]) : lanes_max<G>(v[k]);
    if ((threadIdx.x & 63) < G) s.red[threadIdx.x >> 6][k][p] = v[k];
  }
  __syncthreads();
  if (threadIdx.x < G && on) {
#pragma unroll
    for (int k = 0; k < kStats; ++k)
      for (int w = 1; w < T / 64; ++w)
        v[k] = k < 8 ? v[k] + s.red[w][k][p] : fmax(v[k], s.red[w][k][p]);
    constexpr int kQ = kRecTurns / 4;
    const double e = 1e-6 * emit;
    auto cdiff = [](double a, double b) {
      double d = fabs(a - b);
      d = d - floor(d);
      return fmin(d, 1.0 - d);
    };
    // mean j0 + <d>, variance <d^2> - <d>^2: at least <d>^2 / 1024, since the
    // first turn is itself <d> away, so the difference loses at most ten bits
    auto spread = [&](double j0, double d1, double d2) {
      const double md = d1 / kRecTurns, var = d2 / kRecTurns - md * md;
      return sqrt(var < 0.0 ? 0.0 : var) / ((j0 + md) + e);  // (a NaN stays one)
    };
    const double a0x = sqrt(2.0 * jx0 / emit), a0y = sqrt(2.0 * jy0 / emit);
    const double r0 = sqrt(a0x * a0x + a0y * a0y);
    float* o = out + (size_t)i * kIn;
    o[0] = (float)a0x;
    o[1] = (float)a0y;
    o[2] = (float)r0;
    o[3] = (float)atan2(a0y, a0x);
    o[4] = q[0];
    o[5] = q[1];
    o[6] = q[2];
    o[7] = q[3];
    o[8] = (float)log10(cdiff(q[2], q[0]) + 1e-12);
    o[9] = (float)log10(cdiff(q[3], q[1]) + 1e-12);
    o[10] = (float)((v[3] / kQ + e) / (v[2] / kQ + e) - 1.0);
    o[11] = (float)((v[7] / kQ + e) / (v[6] / kQ + e) - 1.0);
    o[12] = (float)spread(jx0, v[0], v[1]);
    o[13] = (float)spread(jy0, v[4], v[5]);
    o[14] = (float)(sqrt(v[8]) / r_ap);
    o[15] = (float)((2.0 * v[9] / emit) / (r0 * r0 + 1e-6));
  }
}

// Column mean and 1/std of features over rows with mask != 0 (one workgroup,
// fixed reduction order): thread t holds columns 4 (t % 4) .. + 3 of rows
// t / 4, t / 4 + 256, ... (a wave reads 16 rows, 1 KB, at once, eight rows of a
// thread in flight), then the sums are reduced pairwise; norm = [mean[16],
// inv_std[16]].  What bounds it: one CU's reads (a second workgroup would
// need memory for its sums, which this call is not given): 0.64 ms for 2^20
// rows, 105 GB/s; 2.06 ms when a thread read whole rows one after the other.
__global__ void __launch_bounds__(1024) k_feature_stats(const float* __restrict__ f,
                                                        const int32_t* __restrict__ mask,
                                                        int64_t n, float* __restrict__ norm) {
  __shared__ double acc[9][1024];
  const int c4 = threadIdx.x & 3;
  double s1[4] = {}, s2[4] = {}, cnt = 0.0;
  auto add = [&](const float (&v)[4]) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const double d = v[c];
      s1[c] += d;
      s2[c] = fma(d, d, s2[c]);  // the square is exact
    }
    cnt += 1.0;
  };
  constexpr int kRows = 256, kAhead = 8;
  int64_t i = threadIdx.x >> 2;
  if (!mask) {
    for (; i + (kAhead - 1) * kRows < n; i += kAhead * kRows) {
      float v[kAhead][4];
#pragma unroll
      for (int k = 0; k < kAhead; ++k)
#pragma unroll
        for (int c = 0; c < 4; ++c) v[k][c] = f[(i + k * kRows) * 16 + 4 * c4 + c];
#pragma unroll
      for (int k = 0; k < kAhead; ++k) add(v[k]);
    }
  }
  for (; i < n; i += kRows) {
    if (mask && !mask[i]) continue;
    float v[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) v[c] = f[i * 16 + 4 * c4 + c];
    add(v);
  }
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    acc[c][threadIdx.x] = s1[c];
    acc[4 + c][threadIdx.x] = s2[c];
  }
  acc[8][threadIdx.x] = cnt;
  __syncthreads();
  for (int st = 512; st >= 4; st >>= 1) {
    if ((int)threadIdx.x < st)
#pragma unroll
      for (int k = 0; k < 9; ++k) acc[k][threadIdx.x] += acc[k][threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x < 16) {
    const int c = threadIdx.x;
    const double nn = acc[8][0];
    const double m = nn > 0 ? acc[c % 4][c / 4] / nn : 0.0;
    const double var = nn > 0 ? acc[4 + c % 4][c / 4] / nn - m * m : 1.0;
    norm[c] = (float)m;
    norm[16 + c] = (float)(1.0 / sqrt(var > 1e-30 ? var : 1.0));
  }
}

// Retire alive particles whose logit >= threshold unless audited: audited iff
// the first Philox word of (key audit_seed, counter (pid_lo, pid_hi,
// 0xFFFFFFFF, 0)) is below audit_threshold.  Retired particles get state 2.
// counts[0] += retired, counts[1] += audited (alive, eligible by logit);
// audit_flags[p] = 1 for each audited particle when the array is given.
__global__ void __launch_bounds__(256) k_retire(SoA P, const int32_t* __restrict__ idx,
                                                const int32_t* __restrict__ ctrl,
                                                const float* __restrict__ logit,
                                                float threshold, unsigned long long audit_seed,
                                                unsigned int audit_threshold,
                                                unsigned int* __restrict__ counts,
                                                int32_t* __restrict__ audit_flags) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= ctrl[0]) return;
  const int32_t p = idx[i];
  if (P.state[p] != 1) return;
  if (!(logit[p] >= threshold)) return;
  const unsigned long long pid = (unsigned long long)P.pid[p];
  xtmm::U4 c{(unsigned int)pid, (unsigned int)(pid >> 32), 0xFFFFFFFFu, 0u};
  const xtmm::U4 w = xtmm::philox4x32_10(c, (unsigned int)audit_seed,
                                         (unsigned int)(audit_seed >> 32));
  if (w.a < audit_threshold) {
    atomicAdd(&counts[1], 1u);
    if (audit_flags) audit_flags[p] = 1;
    return;
  }
  P.state[p] = 2;
  atomicAdd(&counts[0], 1u);
}

// Score of the retire rule without the network: -max(f8, f9), the larger of
// the two tune-diffusion features negated (a NaN feature gives a NaN score,
// which no threshold retires).
__global__ void __launch_bounds__(256) k_rule_score(const float* __restrict__ f, int64_t n,
                                                    float* __restrict__ score) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float a = f[i * kIn + 8], b = f[i * kIn + 9];
  score[i] = (a != a || b != b) ? __builtin_nanf("") : -(a > b ? a : b);
}

// ------------------------------------------------------------- launchers
hipError_t launch_mlp_forward(const float* theta, const float* norm, const float* X, int64_t B,
                              float* logit, hipStream_t s) {
  if (B <= 0) return hipSuccess;
  // four tiles a wave once that still gives every CU a block (2^16 rows: 256
  // blocks), one before; at most the two blocks per CU that are resident at once,
  // each of which loads the network once (1,024 blocks: 66 us for 2^20 rows, 512: 63,
  // before the activation moved between the products).  us a call for 16,384 /
  // 2^17 / 2^20 rows: 13 / 10.5 / 55 (29 / 108 / 757 with one block per 64 rows and
  // the staging of every operand).
  if (B >= 65536) {
    const int64_t nb = (B + 255) / 256;
    hipLaunchKernelGGL(k_mlp_forward<4>, dim3((unsigned)(nb < 512 ? nb : 512)), dim3(256), 0, s,
                       theta, norm, X, B, logit);
  } else {
    hipLaunchKernelGGL(k_mlp_forward<1>, dim3((unsigned)((B + 63) / 64)), dim3(256), 0, s, theta,
                       norm, X, B, logit);
  }
  return hipGetLastError();
}

int64_t mlp_workspace_floats(int64_t B) {
  const int64_t nb = (B + kSamplesPerBlock - 1) / kSamplesPerBlock;
  return nb * (kParams + 1);
}

// Workspace of the allocation-free gradient entry point (batches of at most
// kMlpNoAllocMaxBatch rows).  Every launch of k_mlp_grad writes all the
// partials the reduction then reads, so the array never needs clearing.  In
// host code `scratch` names a host-side stand-in: kernels receive the device
// address looked up below, never the symbol itself.
constexpr int64_t kNoAllocFloats =
    ((kMlpNoAllocMaxBatch + kSamplesPerBlock - 1) / kSamplesPerBlock) * (kParams + 1);
static __device__ __align__(256) float scratch[kNoAllocFloats];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
float* g_scratch_addr[kMaxDevices] = {};
}  // namespace

hipError_t mlp_noalloc_workspace(float** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_addr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_addr[dev] = static_cast<float*>(p);
  }
  *out = g_scratch_addr[dev];
  return hipSuccess;
}

namespace {
// column splits of a 64-row block: as many as keep the launch within one block
// per CU (256), of 1, 2, 4
unsigned grad_split(int64_t nb) { return nb <= 64 ? 4u : (nb <= 128 ? 2u : 1u); }

void enqueue_grad(const float* theta, const float* norm, const float* X, const float* Y,
                  const int32_t* perm, int64_t B, float pos_weight, float* work, hipStream_t s) {
  const int64_t nb = (B + kSamplesPerBlock - 1) / kSamplesPerBlock;
  hipLaunchKernelGGL(k_mlp_grad, dim3((unsigned)nb, grad_split(nb)), dim3(256), 0, s, theta, norm,
                     X, Y, perm, B, pos_weight, work, work + (size_t)nb * kParams);
}

constexpr unsigned kParamBlocks = (kParams + 1 + 63) / 64;  // one thread more: the loss
}  // namespace

hipError_t launch_mlp_grad(const float* theta, const float* norm, const float* X, const float* Y,
                           int64_t B, float pos_weight, float* grad, float* loss, float* work,
                           hipStream_t s) {
  if (B <= 0) return hipSuccess;
  const int nb = (int)((B + kSamplesPerBlock - 1) / kSamplesPerBlock);
  enqueue_grad(theta, norm, X, Y, nullptr, B, pos_weight, work, s);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_mlp_reduce, dim3(kParamBlocks), dim3(64), 0, s, work, nb,
                     work + (size_t)nb * kParams, grad, loss, B);
  return hipGetLastError();
}

hipError_t launch_adam(float* theta, float* m, float* v, const float* grad, int32_t step, float lr,
                       hipStream_t s) {
  hipLaunchKernelGGL(k_adam, dim3(kParamBlocks), dim3(64), 0, s, theta, m, v, grad,
                     step, lr);
  return hipGetLastError();
}

hipError_t launch_adam_bias(double2* bias, int32_t first_step, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_adam_bias, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, bias,
                     first_step, (int)n);
  return hipGetLastError();
}

hipError_t launch_mlp_train_step(float* theta, float* m, float* v, const float* norm,
                                 const float* X, const float* Y, const int32_t* perm, int64_t B,
                                 float pos_weight, const double2* bias, float lr, float* loss,
                                 float* work, hipStream_t s) {
  if (B <= 0) return hipSuccess;
  const int nb = (int)((B + kSamplesPerBlock - 1) / kSamplesPerBlock);
  enqueue_grad(theta, norm, X, Y, perm, B, pos_weight, work, s);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_mlp_reduce_adam, dim3(kParamBlocks), dim3(64), 0, s, work, nb,
                     work + (size_t)nb * kParams, loss, B, theta, m, v, bias, lr);
  return hipGetLastError();
}

hipError_t launch_mlp_init(float* theta, unsigned long long seed, hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_init, dim3((kParams + 255) / 256), dim3(256), 0, s, theta, seed);
  return hipGetLastError();
}

hipError_t launch_features(const float* rec, int64_t n, const double twiss4[4], double emit,
                           double r_ap, const float2* tw, const float* win, float* out,
                           hipStream_t s) {
  if (n <= 0) return hipSuccess;
  // Eight particles in 512 threads; four in 256 while that is at most one
  // workgroup per CU (256 CUs).  us for 500 / 2,000 / 20,000 / 100,000
  // particles: 4 in 256 threads 24 / 33 / 208 / 928, 8 in 512 27 / 30 / 192 /
  // 921, 16 in 512 46 / 57 / 224 / 1,007, 16 in 1,024 41 / 46 / 255 / 1,258.
  auto launch = [&](auto kernel, int64_t g, int t) {
    const int64_t groups = (n + g - 1) / g;
    hipLaunchKernelGGL(kernel, dim3((unsigned)((groups + 7) / 8 * 8)), dim3(t), 0, s, rec, n,
                       twiss4[0], twiss4[1], twiss4[2], twiss4[3], emit, r_ap, tw, win, out);
  };
  if (n >= (int64_t)1 << 22) launch(k_features<8, 512, uint64_t>, 8, 512);
  else if (n > 1024) launch(k_features<8, 512, uint32_t>, 8, 512);
  else launch(k_features<4, 256, uint32_t>, 4, 256);
  return hipGetLastError();
}

hipError_t launch_feature_stats(const float* f, const int32_t* mask, int64_t n, float* norm,
                                hipStream_t s) {
  hipLaunchKernelGGL(k_feature_stats, dim3(1), dim3(1024), 0, s, f, mask, n, norm);
  return hipGetLastError();
}

hipError_t launch_retire(SoA P, const int32_t* idx, const int32_t* ctrl, int64_t grid_upper,
                         const float* logit, float threshold, unsigned long long audit_seed,
                         unsigned int audit_threshold, unsigned int* counts, int32_t* audit_flags,
                         hipStream_t s) {
  if (grid_upper <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_retire, dim3((unsigned)((grid_upper + 255) / 256)), dim3(256), 0, s, P, idx,
                     ctrl, logit, threshold, audit_seed, audit_threshold, counts, audit_flags);
  return hipGetLastError();
}

hipError_t launch_rule_score(const float* f, int64_t n, float* score, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_rule_score, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, f, n, score);
  return hipGetLastError();
}

}  // namespace xtm
