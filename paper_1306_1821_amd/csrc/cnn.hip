// 3-D CNN of the learned warm start and mass (include/cnn.h) on gfx950 MFMA.
//
// Every 3x3x3 convolution is an implicit GEMM on 16x16x16 bf16 MFMA tiles
// (float32 accumulation): 16 output channels (rows) by 16 consecutive voxels
// (columns); the K loop runs over (tap, input channel).
// Activations are channels-last bfloat16 [V][4] (input, 3 channels + zero
// pad) or [V][16]; pre-activations float32 [V][16], [V][2] for the last layer.
// Lane layout of the MFMA (lane l, element i): A[l % 16][4 (l / 16) + i],
// B[4 (l / 16) + i][l % 16], D[4 (l / 16) + i][l % 16].
//
// Backward: the input gradient is the same convolution of the output gradient
// with mirrored taps and transposed weights, fused with GELU'(z); the weight
// gradient runs the MFMA with K over voxels (A = activations gathered per tap,
// B = output gradient), one partial per block, summed in a fixed order.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>
#include <vector>

#include "../../include/cnn.h"

namespace cnnk {

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kCin[4] = {3, 16, 16, 16};
constexpr int kCout[4] = {16, 16, 16, 2};
constexpr int kTile = 27 * 256;  // entries of one weight-gradient partial
// weight-gradient partials at most: 3 blocks on each of 256 compute units, and the same number
// on a device (partition) with fewer, so that a gradient's rounding does not depend on it
constexpr int kParts = 768;

inline int off_w(int l) {
  int o = 0;
  for (int k = 0; k < l; ++k) o += 27 * kCin[k] * kCout[k] + kCout[k];
  return o;
}
inline int off_b(int l) { return off_w(l) + 27 * kCin[l] * kCout[l]; }
inline int n_params() { return off_w(4); }
// past the gradient, the last layer's bias padded to 16 channels (16-byte aligned)
inline int off_pad() { return (n_params() + 3) / 4 * 4; }
inline int n_grad() { return off_pad() + 16; }

__device__ __forceinline__ uint16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }
// GELU(z) = z Phi(z) with the normal CDF written as Phi(z) = erfc(-z / sqrt 2) / 2,
// which keeps its relative accuracy in the lower tail (1 + erf(.) cancels there)
__device__ __forceinline__ float norm_cdf(float z) { return 0.5f * erfcf(-z * 0.70710678118654752f); }
__device__ __forceinline__ float gelu(float z) { return z * norm_cdf(z); }
__device__ __forceinline__ float gelu_grad(float z) {
  return norm_cdf(z) + z * expf(-0.5f * z * z) * 0.3989422804014327f;
}

// The same GELU and GELU' values rounded to bf16, four at a time and bit for bit, without
// erfcf where the rounding does not need its last digits.  With y = |z| and t = 1 / (1 + 0.3 y),
//   Phi(-y) = exp(-y^2 / 2) t P(t),
// P the degree-7 polynomial with the smallest relative error on 0 <= y <= 10.5 (5.0e-8, 7.5e-8
// with its coefficients rounded to float32; a weighted least-squares fit iterated towards equal
// ripples).  Evaluated in float32 the value is
// within kErr0 + kErr1 y^2 (relative; for GELU' times the magnitudes of the two terms it
// adds) of the erfcf form above; where no bf16 rounding boundary lies within that distance,
// both round to the same bf16 value, else (about one value in 950), and outside the range of
// the bound (y >= 10, tiny, huge or not finite), the erfcf form decides.  cnn_gelu_check
// compares the two: no value differs, and the largest deviation is 0.53 of the bound for GELU at
// every float32 z, 0.73 for v GELU'(z) at every z with v = 1 and three random v.  erfcf is about 50
// instructions, three of them quarter rate, and at 256^3 a layer evaluates it 268 million
// times: a hidden layer went from 713 to 562 us and the first from 511 to 380 us.
constexpr float kErr0 = 9e-7f, kErr1 = 3.75e-7f;
struct Cdf {
  float q, e, y2;  // Phi(-|z|), exp(-z^2 / 2), z^2
};
__device__ __forceinline__ Cdf norm_cdf_short(float z) {
  const float t = __builtin_amdgcn_rcpf(__builtin_fmaf(0.3f, fabsf(z), 1.f));
  float p = 0.037548013f;
  p = __builtin_fmaf(p, t, -0.165077418f);
  p = __builtin_fmaf(p, t, 0.220085055f);
  p = __builtin_fmaf(p, t, -0.0665243194f);
  p = __builtin_fmaf(p, t, 0.135496393f);
  p = __builtin_fmaf(p, t, 0.097756058f);
  p = __builtin_fmaf(p, t, 0.121111214f);
  p = __builtin_fmaf(p, t, 0.119605042f);
  Cdf c;
  c.y2 = z * z;
  c.e = __builtin_amdgcn_exp2f(-0.721347520444481704f * c.y2);
  c.q = c.e * (t * p);
  return c;
}
// true if r - b and r + b (b >= 0) round to the same bf16 value
__device__ __forceinline__ bool same_bf(float r, float b) {
  return ((__float_as_uint(r - b) + 0x8000u) ^ (__float_as_uint(r + b) + 0x8000u)) < 0x10000u;
}
__device__ __forceinline__ bool plain(float r) { return fabsf(r) > 1e-30f && fabsf(r) < 1e30f; }

// GELU(z) = max(z, 0) - |z| Phi(-|z|), and whether z is in the range of its bound
__device__ __forceinline__ float gelu_short(float z, const Cdf& c) {
  return __builtin_fmaf(-fabsf(z), c.q, fmaxf(z, 0.f));
}
__device__ __forceinline__ bool gelu_short_in(const Cdf& c) {
  // 1e-12 < z^2 < 100 (as integers; also false for NaN)
  return __float_as_uint(c.y2) - 0x2b8cbcccu < 0x42c80000u - 0x2b8cbcccu;
}
// the bound in units of the last place, which is at most 2^-23 of the value
__device__ __forceinline__ float gelu_short_ulps(const Cdf& c) {
  return __builtin_fmaf(kErr1 * 16777216.f, c.y2, kErr0 * 16777216.f);
}
// v GELU'(z) = v (phi + zp) and its bound
struct GradShort {
  float phi, err, zp;
  __device__ __forceinline__ GradShort(float z, const Cdf& c)
      : phi(z > 0.f ? 1.f - c.q : c.q), err(__builtin_fmaf(kErr1, c.y2, kErr0)), zp(z * (c.e * 0.3989422804014327f)) {}
  __device__ __forceinline__ float value(float v) const { return v * (phi + zp); }
  __device__ __forceinline__ float bound(float v) const { return fabsf(v) * (err * (phi + fabsf(zp))); }
};

// rounded GELU: the distance of the low 16 bits from a rounding boundary against the bound
__device__ __forceinline__ ushort4 gelu_bf4(const float* z) {
  uint16_t o[4];
  bool ok[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const Cdf c = norm_cdf_short(z[i]);
    const uint32_t u = __float_as_uint(gelu_short(z[i], c));
    const float d = (float)(int)(int16_t)(uint16_t)(u ^ 0x8000u);
    ok[i] = gelu_short_in(c) && fabsf(d) > gelu_short_ulps(c);
    o[i] = (uint16_t)((u + 0x8000u) >> 16);
  }
  if (!(ok[0] && ok[1] && ok[2] && ok[3])) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (!ok[i]) o[i] = f2bf(gelu(z[i]));
  }
  return make_ushort4(o[0], o[1], o[2], o[3]);
}
// v gelu'(z)
__device__ __forceinline__ ushort4 gelu_grad_bf4(const float* v, const float* z) {
  uint16_t o[4];
  bool ok[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const Cdf c = norm_cdf_short(z[i]);
    const GradShort g(z[i], c);
    const float r = g.value(v[i]);
    ok[i] = c.y2 < 100.f && plain(r) && same_bf(r, g.bound(v[i]));
    o[i] = (uint16_t)((__float_as_uint(r) + 0x8000u) >> 16);
  }
  if (!(ok[0] && ok[1] && ok[2] && ok[3])) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (!ok[i]) o[i] = f2bf(v[i] * gelu_grad(z[i]));
  }
  return make_ushort4(o[0], o[1], o[2], o[3]);
}

// ------------------------------------------------------------------ kernels
__global__ void __launch_bounds__(256) k_features(long long nv, const float* __restrict__ beta,
                                                  float scale, const float* __restrict__ mask,
                                                  const float* __restrict__ sel,
                                                  float* __restrict__ out3) {
  for (long long v = (long long)blockIdx.x * 256 + threadIdx.x; v < nv; v += (long long)gridDim.x * 256) {
    out3[v] = beta[v] * scale;
    out3[nv + v] = mask[v];
    out3[2 * nv + v] = sel[v];
  }
}

enum ConvMode : int { C_FWD_GELU = 0, C_FWD_LAST = 1, C_DGRAD = 2 };

// Bricks of the convolutions: 4 x CY x 16 voxels (x, y, z) with a one-voxel halo, staged
// in LDS; every grid side is a multiple of 4, so only y and z can overhang.
constexpr int kCX = 4, kBZ = 16;
constexpr int kCHX = kCX + 2, kHZ = kBZ + 2;

__host__ __device__ inline int conv_bricks(int n, int cy) {
  return (n / kCX) * ((n + cy - 1) / cy) * ((n + kBZ - 1) / kBZ);
}

// Workgroups are dealt to the 8 XCDs round-robin; brick_of gives each XCD a contiguous
// run of bricks, so that neighbours (which share their halos) meet in one L2.
__device__ __forceinline__ int brick_of(int b, int g) {
  const int q = g >> 3, r = g & 7, x = b & 7, i = b >> 3;
  return x < r ? x * (q + 1) + i : r * (q + 1) + (x - r) * q + i;
}

// One 3x3x3 convolution (zero padding).  Wave w of a block owns the brick's x plane w: CY
// rows (8, or 2 on small grids, see conv_rows) of 16 z voxels, one accumulator tile each; the
// counts below are for 8.  The weights are the MFMA's A operand
// (rows = output channels) and a row's shifted activations its B operand (columns =
// voxels), so a lane ends up with 4 consecutive output channels of one voxel and stores
// them together (64 lanes cover 16 whole voxels; with the operands the other way round a
// store wrote 2 bytes per lane).  K runs over taps, 16 channels at a time (CS = 16), or 4
// taps x 4 channels (CS = 4: the network's input, read as float32 and rounded here).  A
// fragment read from LDS serves every row of the wave that needs it (up to 3 of the 8):
// 90 reads for 216 MFMAs, where one read per MFMA kept LDS as busy as the matrix cores.  The
// two halves of the channels lie in separate planes of the brick, so that half a wave
// (16 voxels x 8 channels) reads 256 bytes in a row (whole voxels of 32 bytes met every bank
// twice: LDS was busy for 322 us of the last layer at 256^3, which went from 432 to 394 us).
// The order of the products of one output is the same for every brick and voxel: that of
// the taps, except in the last layer outside training.  That one has two output channels,
// which leaves 14 of the 16 matrix rows empty: its rows are (y tap, channel), one accumulator
// tile for each of the 10 haloed rows, and K is 32, two taps of 16 channels at once (a lane
// reads the 8 channels of one plane of the brick): 50 MFMAs and 50 reads a wave instead of
// 216 and 90; an output is the sum of three rows of three tiles.  Its float32 sums take
// another order for that.  Training keeps the order of the taps: the output gradient is
// rounded to bfloat16, and the small differences that come of it grow from step to step
// (14 of 924 us at 128^3); so do the hidden layers, whose results are rounded as well.
// What bounds it at 256^3: for the hidden layers the products, GELU and the stores (570 us;
// 763 before this form and the short GELU), for the last layer the staging (289 us;
// 382 with its two channels as rows, 661 plus 257 us to pick its two channels out of 16
// before that).  A forward at 256^3 went from 1648 to 1540 us with the last layer's form.
// TRAIN: keep the pre-activation for the backward pass.  LAST: out0, out1 are the two
// output channels, or out0 the pairs [V][2] for the loss (TRAIN).
template <int CS, int MODE, bool TRAIN, int CY>
__global__ void __launch_bounds__(256, 4) k_conv(int n, const void* __restrict__ in,
                                                 const bf16x4* __restrict__ wp,
                                                 const float* __restrict__ bias,
                                                 const float* __restrict__ zprev,
                                                 float* __restrict__ out0, float* __restrict__ out1,
                                                 uint16_t* __restrict__ aout) {
  constexpr int kCHY = CY + 2, kCHalo = kCHX * kCHY * kHZ;  // voxels of the haloed brick
  constexpr int kItems = CS == 16 ? 2 * kCHalo : kCHalo;  // 16-byte halves / whole voxels
  constexpr int kIter = (kItems + 255) / 256;
  __shared__ uint4 brick[CS == 16 ? 2 * kCHalo : kCHalo / 2];  // [channel half][voxel] / [voxel][4]
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int nbz = (n + kBZ - 1) / kBZ, nby = (n + CY - 1) / CY;
  const int bk = brick_of(blockIdx.x, gridDim.x);
  const int x0 = bk / (nbz * nby) * kCX, y0 = bk / nbz % nby * CY, z0 = bk % nbz * kBZ;
  const long long nv = (long long)n * n * n;
  // stage the brick with its halo (zeros outside the grid), every load first
  uint4 st[CS == 16 ? kIter : 1];
  float sf[CS == 16 ? 1 : kIter][3];
#pragma unroll
  for (int k = 0; k < kIter; ++k) {
    const int i = threadIdx.x + 256 * k, vox = CS == 16 ? i >> 1 : i;
    const int xx = x0 + vox / (kHZ * kCHY) - 1, yy = y0 + vox / kHZ % kCHY - 1, zz = z0 + vox % kHZ - 1;
    const bool ok = i < kItems && (unsigned)xx < (unsigned)n && (unsigned)yy < (unsigned)n && (unsigned)zz < (unsigned)n;
    const long long v = ((long long)xx * n + yy) * n + zz;
    if constexpr (CS == 16) {
      st[k] = make_uint4(0u, 0u, 0u, 0u);
      if (ok) st[k] = reinterpret_cast<const uint4*>(in)[2 * v + (i & 1)];
    } else {
#pragma unroll
      for (int c = 0; c < 3; ++c) sf[k][c] = ok ? reinterpret_cast<const float*>(in)[c * nv + v] : 0.f;
    }
  }
  constexpr bool kPairs = MODE == C_FWD_LAST && !TRAIN;  // two taps a product
  constexpr int NC = kPairs ? 1 : CS == 16 ? 27 : 7;
  bf16x4 w[NC];
  bf16x4 w2[kPairs ? 4 : 1][2];
  if constexpr (kPairs) {  // matrix row 2 dy + channel, from wp's row of that channel
    const int dy = (lane & 15) >> 1, at = dy * 3 * 64 + (lane & 1), g = lane >> 4;
    const bf16x4 none = {0, 0, 0, 0};
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int tap = c < 3 ? 9 * c + (g >> 1) : 9 * (g >> 1) + 2;
#pragma unroll
      for (int h = 0; h < 2; ++h) w2[c][h] = dy < 3 ? wp[tap * 64 + at + (2 * (g & 1) + h) * 16] : none;
    }
    w[0] = dy < 3 ? wp[20 * 64 + at + g * 16] : none;
  } else {
#pragma unroll
    for (int c = 0; c < NC; ++c) w[c] = wp[c * 64 + lane];
  }
#pragma unroll
  for (int k = 0; k < kIter; ++k) {
    const int i = threadIdx.x + 256 * k;
    if (i < kItems) {
      if constexpr (CS == 16)
        brick[(i & 1) * kCHalo + (i >> 1)] = st[k];
      else
        reinterpret_cast<ushort4*>(brick)[i] = make_ushort4(f2bf(sf[k][0]), f2bf(sf[k][1]), f2bf(sf[k][2]), 0);
    }
  }
  __syncthreads();
  const int m = lane & 15, grp = lane >> 4;
  const bf16x4* lb = reinterpret_cast<const bf16x4*>(brick);
  const int ofs = (grp >> 1) * 2 * kCHalo + (grp & 1);  // the lane's 4 channels (CS = 16)
  constexpr int kRows = kPairs ? kCHY : CY;
  f32x4 acc[kRows];
#pragma unroll
  for (int r = 0; r < kRows; ++r) acc[r] = f32x4{0.f, 0.f, 0.f, 0.f};
  if constexpr (kPairs) {
    // tap pairs (dz 0, 1) of each dx, then dz = 2 of dx 0, 1; a lane reads 8 channels of one
    const int half = (grp & 1) * kCHalo, second = grp >> 1;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int at = c < 3 ? (wave + c) * kCHY * kHZ + m + second : (wave + second) * kCHY * kHZ + m + 2;
      const bf16x8 a = __builtin_bit_cast(bf16x8, __builtin_shufflevector(w2[c][0], w2[c][1], 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
      for (int hy = 0; hy < kCHY; ++hy)
        acc[hy] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
            a, __builtin_bit_cast(bf16x8, brick[half + at + hy * kHZ]), acc[hy], 0, 0, 0);
    }
#pragma unroll
    for (int hy = 0; hy < kCHY; ++hy)  // dx = 2, dz = 2
      acc[hy] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(
          w[0], lb[(((wave + 2) * kCHY + hy) * kHZ + m + 2) * 2 + ofs], acc[hy], 0, 0, 0);
    // rows (dy, channel): dy 0 and 1 in the lanes of group 0, dy 2 in those of group 1
#pragma unroll
    for (int r = 0; r < CY; ++r)
#pragma unroll
      for (int o = 0; o < 2; ++o)
        acc[r][o] = (acc[r][o] + acc[r + 1][2 + o]) + __shfl_xor(acc[r + 2][o], 16);
  } else if constexpr (CS == 16) {
#pragma unroll
    for (int dx = 0; dx < 3; ++dx)
#pragma unroll
      for (int hy = 0; hy < kCHY; ++hy)
#pragma unroll
        for (int dz = 0; dz < 3; ++dz) {
          const bf16x4 b = lb[(((wave + dx) * kCHY + hy) * kHZ + m + dz) * 2 + ofs];
#pragma unroll
          for (int r = 0; r < CY; ++r)
            if (r <= hy && hy <= r + 2)
              acc[r] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(w[(dx * 3 + hy - r) * 3 + dz], b, acc[r], 0, 0, 0);
        }
  } else {
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int tap = 4 * c + grp;
      const int at = tap < 27 ? (tap / 9 * kCHY + tap / 3 % 3) * kHZ + tap % 3 : 0;
#pragma unroll
      for (int r = 0; r < CY; ++r) {
        bf16x4 b = lb[(wave * kCHY + r) * kHZ + m + at];
        if (c == NC - 1 && tap >= 27) b = bf16x4{0, 0, 0, 0};
        acc[r] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(w[c], b, acc[r], 0, 0, 0);
      }
    }
  }
  float4 bi = make_float4(0.f, 0.f, 0.f, 0.f);
  if (MODE != C_DGRAD) bi = *reinterpret_cast<const float4*>(bias + 4 * grp);
  const int zz = z0 + m;
#pragma unroll
  for (int r = 0; r < CY; ++r) {
    if (y0 + r >= n || zz >= n) continue;
    const long long v = ((long long)(x0 + wave) * n + y0 + r) * n + zz;
    const float val[4] = {acc[r][0] + bi.x, acc[r][1] + bi.y, acc[r][2] + bi.z, acc[r][3] + bi.w};
    if constexpr (MODE == C_FWD_GELU) {
      if (TRAIN) reinterpret_cast<float4*>(out0)[v * 4 + grp] = make_float4(val[0], val[1], val[2], val[3]);
      reinterpret_cast<ushort4*>(aout)[v * 4 + grp] = gelu_bf4(val);
    } else if constexpr (MODE == C_FWD_LAST) {
      if (grp == 0) {  // channels 0, 1
        if (TRAIN) {
          reinterpret_cast<float2*>(out0)[v] = make_float2(val[0], val[1]);
        } else {
          if (out0) out0[v] = val[0];
          if (out1) out1[v] = val[1];
        }
      }
    } else {
      const float4 zv = reinterpret_cast<const float4*>(zprev)[v * 4 + grp];
      const float da[4] = {acc[r][0], acc[r][1], acc[r][2], acc[r][3]}, zp[4] = {zv.x, zv.y, zv.z, zv.w};
      reinterpret_cast<ushort4*>(aout)[v * 4 + grp] = gelu_grad_bf4(da, zp);
    }
  }
}

// Gaussian NLL per voxel; writes the bf16 output gradient [V][16] and block partials.
__global__ void __launch_bounds__(256) k_loss(long long nv, const float2* __restrict__ z4,
                                              const float* __restrict__ target,
                                              uint4* __restrict__ dz4, double* __restrict__ part) {
  __shared__ double red[4];
  double acc = 0.0;
  const float inv = 1.f / (float)nv;
  for (long long v = (long long)blockIdx.x * 256 + threadIdx.x; v < nv; v += (long long)gridDim.x * 256) {
    const float2 out = z4[v];
    const float mu = out.x, s = out.y;
    const float d = target[v] - mu, e = expf(-s);
    acc += 0.5 * ((double)d * d * e + s);
    uint4* o = dz4 + v * 2;
    o[0] = make_uint4(f2bf(-d * e * inv) | (uint32_t)f2bf(0.5f * (1.f - d * d * e) * inv) << 16, 0u, 0u, 0u);
    o[1] = make_uint4(0u, 0u, 0u, 0u);
  }
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) part[blockIdx.x] = ((red[0] + red[1]) + red[2]) + red[3];
}

// Weight gradient: dW[t][ci][co] = sum_v a[v + d_t][ci] dz[v][co], the MFMA's K over 16
// voxels of a z row (B = dz, columns co).  A block walks bricks of BX x BY x 16 voxels and
// stages them channel-major in LDS, the activations with their halo; a staging thread turns
// 4 voxels x 4 channels (8-byte loads and LDS writes).  The channel pitches are an odd
// multiple of 4 words, so that half a wave's fragment reads (16 channels x 2 voxel quads of
// 2 words) meet every one of the 64 banks once.  Wave w owns 4 rows; an input row is read once (an aligned quad and the two voxels
// after it) and gives the fragments of all three z shifts in registers for every row of the
// wave it is a neighbour of: 36 reads for 108 MFMAs, where each fragment took four 2-byte
// reads.  CS = 16: A rows are the input channels of one tap.  CS = 4: A rows are (z shift,
// channel), 9 MFMAs a row instead of 27, read from the network's float32 input.  The
// waves' sums meet in LDS, one partial per block, summed by k_wreduce in a fixed order.
// 128^3: 72 us a 16-channel layer and 66 us for the first (103 and 202 us before); the
// accumulators (108 registers) leave 3 blocks per compute unit.
constexpr int kBX = 2, kBY = 8;
constexpr int kHX = kBX + 2, kHY = kBY + 2, kRowP = 20;  // halo rows hold 18 voxels of 20
constexpr int kChA = kHX * kHY * kRowP + 8, kChD = kBX * kBY * kBZ + 8;  // channel pitches
static_assert(kChA / 2 % 8 == 4 && kChD / 2 % 8 == 4 && kChA % 4 == 0, "channel pitches");

// 4 channels of 4 voxels -> 4 voxels of 4 channels
__device__ __forceinline__ void turn4(const uint2* v, uint2* c) {
  c[0] = make_uint2((v[0].x & 0xffffu) | v[1].x << 16, (v[2].x & 0xffffu) | v[3].x << 16);
  c[1] = make_uint2(v[0].x >> 16 | (v[1].x & 0xffff0000u), v[2].x >> 16 | (v[3].x & 0xffff0000u));
  c[2] = make_uint2((v[0].y & 0xffffu) | v[1].y << 16, (v[2].y & 0xffffu) | v[3].y << 16);
  c[3] = make_uint2(v[0].y >> 16 | (v[1].y & 0xffff0000u), v[2].y >> 16 | (v[3].y & 0xffff0000u));
}

__host__ __device__ inline int wgrad_bricks(int n) {
  return (n / kBX) * ((n + kBY - 1) / kBY) * ((n + kBZ - 1) / kBZ);
}

template <int CS>
__global__ void __launch_bounds__(256, 3) k_wgrad(int n, const void* __restrict__ in,
                                               const uint16_t* __restrict__ dz,
                                               float* __restrict__ part, float* __restrict__ dbpart) {
  constexpr int kT = CS == 16 ? 27 : 9;  // accumulator tiles
  constexpr int kLds = (CS == 16 ? 16 : 3) * kChA + 16 * kChD;
  static_assert(kBX * kBY == 16 && 2 * kLds >= 4 * kT * 256, "rows per wave; reduction buffer");
  __shared__ __align__(16) uint16_t lds[kLds];
  __shared__ float sdb[4][16];
  uint16_t* const sa = lds;
  uint16_t* const sd = lds + (CS == 16 ? 16 : 3) * kChA;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int m = lane & 15, grp = lane >> 4;
  const int nbz = (n + kBZ - 1) / kBZ, nby = (n + kBY - 1) / kBY, nbricks = wgrad_bricks(n);
  const long long nv = (long long)n * n * n;
  f32x4 acc[kT];
#pragma unroll
  for (int t = 0; t < kT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
  float db = 0.f;
  for (int brick = blockIdx.x; brick < nbricks; brick += gridDim.x) {
    const int x0 = brick / (nbz * nby) * kBX, y0 = brick / nbz % nby * kBY, z0 = brick % nbz * kBZ;
    __syncthreads();  // the previous brick's reads are done
    if constexpr (CS == 16) {
      for (int i = tid; i < kHX * kHY * 5 * 4; i += 256) {
        const int cg = i & 3, q = (i >> 2) % 5, row = i / 20;
        const int xx = x0 + row / kHY - 1, yy = y0 + row % kHY - 1, zb = z0 + 4 * q - 1;
        const bool okr = (unsigned)xx < (unsigned)n && (unsigned)yy < (unsigned)n;
        const uint2* src = reinterpret_cast<const uint2*>(in) + (((long long)xx * n + yy) * n + zb) * 4 + cg;
        uint2 v[4], c[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
          v[j] = okr && (unsigned)(zb + j) < (unsigned)n && 4 * q + j < kHZ ? src[4 * j] : make_uint2(0u, 0u);
        turn4(v, c);
#pragma unroll
        for (int j = 0; j < 4; ++j)
          *reinterpret_cast<uint2*>(sa + (4 * cg + j) * kChA + row * kRowP + 4 * q) = c[j];
      }
    } else {
      for (int i = tid; i < kHX * kHY * 5 * 3; i += 256) {
        const int q = i % 5, row = i / 5 % (kHX * kHY), ch = i / (5 * kHX * kHY);
        const int xx = x0 + row / kHY - 1, yy = y0 + row % kHY - 1, zb = z0 + 4 * q - 1;
        const bool okr = (unsigned)xx < (unsigned)n && (unsigned)yy < (unsigned)n;
        const float* src = reinterpret_cast<const float*>(in) + ch * nv + ((long long)xx * n + yy) * n + zb;
        uint32_t v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
          v[j] = okr && (unsigned)(zb + j) < (unsigned)n && 4 * q + j < kHZ ? f2bf(src[j]) : 0u;
        *reinterpret_cast<uint2*>(sa + ch * kChA + row * kRowP + 4 * q) = make_uint2(v[0] | v[1] << 16, v[2] | v[3] << 16);
      }
    }
    {  // one 4 x 4 block of dz per thread
      const int cg = tid & 3, q = (tid >> 2) & 3, row = tid >> 4;
      const int yy = y0 + row % kBY, zb = z0 + 4 * q;
      const uint2* src = reinterpret_cast<const uint2*>(dz) + (((long long)(x0 + row / kBY) * n + yy) * n + zb) * 4 + cg;
      uint2 v[4], c[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = yy < n && zb < n ? src[4 * j] : make_uint2(0u, 0u);  // n % 4 == 0
      turn4(v, c);
#pragma unroll
      for (int j = 0; j < 4; ++j) *reinterpret_cast<uint2*>(sd + (4 * cg + j) * kChD + row * kBZ + 4 * q) = c[j];
    }
    __syncthreads();
    const int rx = wave >> 1, ry0 = (wave & 1) * 4;
    bf16x4 b[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      b[r] = *reinterpret_cast<const bf16x4*>(sd + m * kChD + (wave * 4 + r) * kBZ + 4 * grp);
#pragma unroll
      for (int i = 0; i < 4; ++i) db += bf2f((uint16_t)b[r][i]);
    }
    const uint16_t* sm = sa + (CS == 16 ? m : (m & 3) < 3 ? m & 3 : 2) * kChA + 4 * grp;
#pragma unroll
    for (int dx = 0; dx < 3; ++dx)
#pragma unroll
      for (int h = 0; h < 6; ++h) {
        const uint16_t* p = sm + ((rx + dx) * kHY + ry0 + h) * kRowP;
        const uint2 lo = *reinterpret_cast<const uint2*>(p);
        const uint32_t hi = *reinterpret_cast<const uint32_t*>(p + 4);
        uint2 f[3];  // z shifts 0, 1, 2
        f[0] = lo;
        f[1] = make_uint2(__builtin_amdgcn_alignbit(lo.y, lo.x, 16), __builtin_amdgcn_alignbit(hi, lo.y, 16));
        f[2] = make_uint2(lo.y, hi);
        if constexpr (CS == 16) {
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (r <= h && h <= r + 2)
#pragma unroll
              for (int s = 0; s < 3; ++s) {
                const int t = (dx * 3 + h - r) * 3 + s;
                acc[t] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(bf16x4, f[s]), b[r], acc[t], 0, 0, 0);
              }
        } else {
          const int s = m >> 2;  // 3: rows of no tap, their sums are not read
          const uint2 g = s == 0 ? f[0] : s == 1 ? f[1] : f[2];
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (r <= h && h <= r + 2) {
              const int t = dx * 3 + h - r;
              acc[t] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(bf16x4, g), b[r], acc[t], 0, 0, 0);
            }
        }
      }
  }
  // the four waves' sums, in wave order
  db += __shfl_xor(db, 16);
  db += __shfl_xor(db, 32);
  if (lane < 16) sdb[wave][lane] = db;
  float* const red = reinterpret_cast<float*>(lds);
  for (int w = 0; w < 4; ++w) {
    __syncthreads();
    if (wave == w)
#pragma unroll
      for (int t = 0; t < kT; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          float* o = red + t * 256 + (4 * grp + i) * 16 + m;
          *o = w == 0 ? acc[t][i] : *o + acc[t][i];
        }
  }
  __syncthreads();
  float* o = part + (size_t)blockIdx.x * kTile;
  if constexpr (CS == 16) {
    for (int i = tid; i < kTile; i += 256) o[i] = red[i];
  } else {  // rows (z shift, channel) of (dx, dy) -> rows of tap 3 (dx, dy) + z shift
    for (int i = tid; i < kT * 192; i += 256) {
      const int t = i / 192, row = i / 16 % 12, co = i & 15;
      o[((t * 3 + row / 4) * 16 + row % 4) * 16 + co] = red[t * 256 + row * 16 + co];
    }
  }
  if (tid < 16) dbpart[blockIdx.x * 16 + tid] = ((sdb[0][tid] + sdb[1][tid]) + sdb[2][tid]) + sdb[3][tid];
}

// The short GELU and GELU' against the erfcf forms for the float32 z of 4 groups bit patterns
// from `first` on: out[0], out[1] count bf16 results that differ; the float bits at out + 2 and
// just after are the largest deviations before rounding, relative to the bounds.
__global__ void __launch_bounds__(256) k_gelu_check(uint32_t first, uint32_t groups, uint32_t seed,
                                                    unsigned long long* __restrict__ out) {
  unsigned long long bad = 0, bad_grad = 0;
  float worst = 0.f, worst_grad = 0.f;
  for (uint64_t g = (uint64_t)blockIdx.x * 256 + threadIdx.x; g < groups; g += (uint64_t)gridDim.x * 256) {
    float z[4], v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t bits = first + 4 * (uint32_t)g + i;
      z[i] = __uint_as_float(bits);
      uint32_t h = (bits + 0x9e3779b9u * seed) * 0x85ebca6bu;
      h = (h ^ h >> 15) * 0xc2b2ae35u;
      h ^= h >> 13;
      // seed 0: 1, else a magnitude of 2^-44 .. 2^4 and a sign
      v[i] = seed == 0 ? 1.f : __uint_as_float((h & 0x807fffffu) | (83u + ((h >> 23) & 0xffu) * 48u / 256u) << 23);
    }
    const ushort4 a = gelu_bf4(z), d = gelu_grad_bf4(v, z);
    const uint16_t as[4] = {a.x, a.y, a.z, a.w}, ds[4] = {d.x, d.y, d.z, d.w};
    for (int i = 0; i < 4; ++i) {
      const float want = gelu(z[i]), want_grad = v[i] * gelu_grad(z[i]);
      bad += as[i] != f2bf(want);
      bad_grad += ds[i] != f2bf(want_grad);
      const Cdf c = norm_cdf_short(z[i]);
      if (gelu_short_in(c)) {
        const int ulps = (int)__float_as_uint(gelu_short(z[i], c)) - (int)__float_as_uint(want);
        worst = fmaxf(worst, (float)abs(ulps) / gelu_short_ulps(c));
      }
      const GradShort s(z[i], c);
      const float r = s.value(v[i]);
      if (c.y2 < 100.f && plain(r)) worst_grad = fmaxf(worst_grad, fabsf(r - want_grad) / s.bound(v[i]));
    }
  }
  if (bad) atomicAdd(out, bad);
  if (bad_grad) atomicAdd(out + 1, bad_grad);
  unsigned* w = reinterpret_cast<unsigned*>(out + 2);
  atomicMax(w, __float_as_uint(worst));
  atomicMax(w + 1, __float_as_uint(worst_grad));
}

// One layer's stored state in float32, [V][cout]: pre-activations (rows of zs), bf16
// activations and bf16 pre-activation gradients (either pointer may be null).
__global__ void __launch_bounds__(256) k_layer_state(long long nv, int cout, int zs,
                                                     const float* __restrict__ z16,
                                                     const uint16_t* __restrict__ a16,
                                                     const uint16_t* __restrict__ dz16,
                                                     float* __restrict__ z, float* __restrict__ a,
                                                     float* __restrict__ dz) {
  const long long tot = nv * cout;
  for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < tot; i += (long long)gridDim.x * 256) {
    const long long v = i / cout, ch = i % cout;
    if (z) z[i] = z16[v * zs + ch];
    if (a) a[i] = bf2f(a16[v * 16 + ch]);
    if (dz) dz[i] = bf2f(dz16[v * 16 + ch]);
  }
}

// Sum the per-block partials of one layer into the flat gradient.  A block takes 64
// consecutive entries of the [27][16][16] partial tile and splits the partials over its
// 16 waves (wave s: partials s, s + 16, ...), whose sums it adds in wave order, so the
// order is fixed; the block past the tile does the same for the 16 bias sums.  Reading
// the partials is the bound (768 x 27.6 KB = 21 MB at 128^3: 5.2 us); a thread that walked
// all partials of one entry by itself had one dependent add per 27.6 KB of stride and
// 27 blocks in flight (767 us a layer with 2048 partials).
constexpr int kRedBlocks = kTile / 64;  // and one block more for the biases
__global__ void __launch_bounds__(1024) k_wreduce(const float* __restrict__ part,
                                                  const float* __restrict__ dbpart, int nw, int cin,
                                                  int cout, float* __restrict__ gw, float* __restrict__ gb) {
  __shared__ float red[1024];
  const int tid = threadIdx.x;
  float s = 0.f;
  if (blockIdx.x < kRedBlocks) {
    const float* p = part + blockIdx.x * 64 + (tid & 63);
#pragma unroll 8
    for (int w = tid >> 6; w < nw; w += 16) s += p[(size_t)w * kTile];
  } else {
#pragma unroll 8
    for (int w = tid >> 4; w < nw; w += 64) s += dbpart[w * 16 + (tid & 15)];
  }
  red[tid] = s;
  __syncthreads();
  if (blockIdx.x < kRedBlocks) {
    if (tid >= 64) return;
    const int idx = blockIdx.x * 64 + tid, t = idx >> 8, ci = (idx >> 4) & 15, co = idx & 15;
    s = red[tid];
    for (int k = 1; k < 16; ++k) s += red[64 * k + tid];
    if (ci < cin && co < cout) gw[(t * cin + ci) * cout + co] = s;
  } else if (tid < cout) {
    s = red[tid];
    for (int k = 1; k < 64; ++k) s += red[16 * k + tid];
    gb[tid] = s;
  }
}

__global__ void __launch_bounds__(256) k_adam(int np, float* __restrict__ p, const float* __restrict__ g,
                                              float* __restrict__ m1, float* __restrict__ m2, float lr,
                                              float c1, float c2) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= np) return;
  const float gi = g[i];
  m1[i] = 0.9f * m1[i] + 0.1f * gi;
  m2[i] = 0.999f * m2[i] + 0.001f * gi * gi;
  p[i] -= lr * (m1[i] / c1) / (sqrtf(m2[i] / c2) + 1e-8f);
}

// bf16 MFMA A operands of one layer: forward (wp) and mirrored/transposed (wd).
__global__ void __launch_bounds__(256) k_pack(const float* __restrict__ W, int cin, int cout,
                                              int forward, int nchunk, bf16x4* __restrict__ out) {
  const int idx = blockIdx.x * 256 + threadIdx.x;
  if (idx >= nchunk * 64) return;
  const int c = idx / 64, lane = idx % 64;
  bf16x4 r;
  for (int i = 0; i < 4; ++i) {
    float w = 0.f;
    if (forward) {
      const int co = lane % 16;
      int tap, ci;
      if (cin == 3) {
        tap = 4 * c + lane / 16;
        ci = i;
      } else {
        tap = c;
        ci = 4 * (lane / 16) + i;
      }
      if (tap < 27 && ci < cin && co < cout) w = W[(tap * cin + ci) * cout + co];
    } else {
      const int co = 4 * (lane / 16) + i, ci = lane % 16, tap = 26 - c;
      if (co < cout && ci < cin) w = W[(tap * cin + ci) * cout + co];
    }
    r[i] = (short)f2bf(w);
  }
  out[idx] = r;
}

}  // namespace cnnk

using namespace cnnk;

struct cnn_ctx {
  hipStream_t stream = nullptr;
  std::string err;
  float *p = nullptr, *g = nullptr, *m1 = nullptr, *m2 = nullptr;
  bf16x4* wp[4] = {nullptr, nullptr, nullptr, nullptr};
  bf16x4* wd[4] = {nullptr, nullptr, nullptr, nullptr};
  int steps = 0;
  int n = 0;
  bool grad_valid = false;  // the stored pre-activations and gradients belong to the last
                            // cnn_gradient / cnn_train_step
  // activations for the current N
  uint16_t* a[3] = {nullptr, nullptr, nullptr};
  // bf16 gradient of the loss with respect to each layer's pre-activations, one
  // buffer per layer so that the last backward pass can be inspected
  uint16_t* dz[4] = {nullptr, nullptr, nullptr, nullptr};
  float *z[4] = {nullptr, nullptr, nullptr, nullptr};
  float *wpart = nullptr, *dbpart = nullptr;
  double *lpart = nullptr, *lpart_h = nullptr;
};

namespace {
thread_local std::string g_cerr;

hmc_status cfail(cnn_ctx* c, hmc_status st, const std::string& why) {
  if (c) c->err = why;
  g_cerr = why;
  return st;
}

#define CCHK(c, call)                                                          \
  do {                                                                         \
    hipError_t e_ = (call);                                                    \
    if (e_ != hipSuccess) return cfail(c, HMC_EDEVICE, std::string(#call) + ": " + hipGetErrorString(e_)); \
  } while (0)

int nchunk_fwd(int l) { return l == 0 ? 7 : 27; }

// y rows of a brick: 2 where bricks of 8 rows would be fewer than the 256 compute units (up to
// 48^3), so that a small grid spreads over more of them and a wave's chain of products, GELU and
// stores is a quarter as long.  Forward (us), 8 and 2 rows: 8^3 31.9 and 18.0, 20^3 35.8 and
// 18.6, 32^3 34.1 and 19.3, 48^3 35.8 and 29.1, 64^3 45.0 and 45.1, 128^3 198 and 242 (a brick
// of 2 rows reads its halo for a quarter of the voxels); training steps 20^3 247 and 184, 48^3
// 268 and 244, 128^3 905 and 1064.
int conv_rows(int n) { return conv_bricks(n, 8) < 256 ? 2 : 8; }

hmc_status pack_all(cnn_ctx* c) {
  for (int l = 0; l < 4; ++l) {
    const int nc = nchunk_fwd(l);
    hipLaunchKernelGGL(k_pack, dim3((nc * 64 + 255) / 256), dim3(256), 0, c->stream,
                       c->p + off_w(l), kCin[l], kCout[l], 1, nc, c->wp[l]);
    if (l > 0)
      hipLaunchKernelGGL(k_pack, dim3((27 * 64 + 255) / 256), dim3(256), 0, c->stream,
                         c->p + off_w(l), kCin[l], kCout[l], 0, 27, c->wd[l]);
  }
  CCHK(c, hipGetLastError());
  return HMC_OK;
}

void free_acts(cnn_ctx* c) {
  for (int i = 0; i < 3; ++i) (void)hipFree(c->a[i]);
  for (int i = 0; i < 4; ++i) (void)hipFree(c->z[i]);
  for (int i = 0; i < 4; ++i) (void)hipFree(c->dz[i]);
  for (int i = 0; i < 4; ++i) c->dz[i] = nullptr;
  for (int i = 0; i < 3; ++i) c->a[i] = nullptr;
  for (int i = 0; i < 4; ++i) c->z[i] = nullptr;
  c->n = 0;
}

hmc_status ensure(cnn_ctx* c, int n) {
  if (n < 4 || n % 4 != 0 || n > 512) return cfail(c, HMC_EINVAL, "N must be a multiple of 4 in 4..512");
  if (c->n == n) return HMC_OK;
  free_acts(c);
  const size_t nv = (size_t)n * n * n;
  for (int i = 0; i < 3; ++i) CCHK(c, hipMalloc(&c->a[i], nv * 16 * sizeof(uint16_t)));
  for (int i = 0; i < 4; ++i) CCHK(c, hipMalloc(&c->z[i], nv * (i < 3 ? 16 : 2) * sizeof(float)));
  for (int i = 0; i < 4; ++i) CCHK(c, hipMalloc(&c->dz[i], nv * 16 * sizeof(uint16_t)));
  c->n = n;
  return HMC_OK;
}

template <int CS, int MODE, bool TRAIN, class... Args>
void launch_conv(cnn_ctx* c, int n, Args... args) {
  const int cy = conv_rows(n);
  const dim3 g(conv_bricks(n, cy)), b(256);
  if (cy == 8)
    hipLaunchKernelGGL((k_conv<CS, MODE, TRAIN, 8>), g, b, 0, c->stream, n, args...);
  else
    hipLaunchKernelGGL((k_conv<CS, MODE, TRAIN, 2>), g, b, 0, c->stream, n, args...);
}

// TRAIN: keeps the pre-activations; out0 / out1: see k_conv
template <bool TRAIN>
hmc_status forward_t(cnn_ctx* c, int n, const float* in3, float* mu, float* logvar) {
  launch_conv<4, C_FWD_GELU, TRAIN>(c, n, in3, c->wp[0], c->p + off_b(0), nullptr, c->z[0], nullptr, c->a[0]);
  for (int l = 1; l < 3; ++l)
    launch_conv<16, C_FWD_GELU, TRAIN>(c, n, c->a[l - 1], c->wp[l], c->p + off_b(l), nullptr, c->z[l], nullptr,
                                       c->a[l]);
  // last layer: bias padded to 16 channels (a device copy past the gradient)
  launch_conv<16, C_FWD_LAST, TRAIN>(c, n, c->a[2], c->wp[3], c->g + off_pad(), nullptr, TRAIN ? c->z[3] : mu,
                                     logvar, nullptr);
  CCHK(c, hipGetLastError());
  return HMC_OK;
}
// forward for training (keeps the pre-activations) and for inference
hmc_status forward(cnn_ctx* c, int n, const float* in3) {
  return forward_t<true>(c, n, in3, nullptr, nullptr);
}
hmc_status infer(cnn_ctx* c, int n, const float* in3, float* mu, float* logvar) {
  c->grad_valid = false;  // overwrites the activations of the last gradient evaluation
  return forward_t<false>(c, n, in3, mu, logvar);
}

hmc_status gradient(cnn_ctx* c, int n, const float* in3, const float* target, double* loss) {
  c->grad_valid = false;
  hmc_status st = forward(c, n, in3);
  if (st != HMC_OK) return st;
  const long long nv = (long long)n * n * n;
  hipLaunchKernelGGL(k_loss, dim3(1024), dim3(256), 0, c->stream, nv, (const float2*)c->z[3], target,
                     (uint4*)c->dz[3], c->lpart);
  const int blocks = std::min(wgrad_bricks(n), kParts);
  for (int l = 3; l >= 0; --l) {
    const uint16_t* dz = c->dz[l];
    if (l == 0)
      hipLaunchKernelGGL(k_wgrad<4>, dim3(blocks), dim3(256), 0, c->stream, n, in3, dz, c->wpart,
                         c->dbpart);
    else
      hipLaunchKernelGGL(k_wgrad<16>, dim3(blocks), dim3(256), 0, c->stream, n, c->a[l - 1], dz,
                         c->wpart, c->dbpart);
    hipLaunchKernelGGL(k_wreduce, dim3(kRedBlocks + 1), dim3(1024), 0, c->stream, c->wpart,
                       c->dbpart, blocks, kCin[l], kCout[l], c->g + off_w(l), c->g + off_b(l));
    if (l > 0)
      launch_conv<16, C_DGRAD, true>(c, n, dz, c->wd[l], nullptr, c->z[l - 1], nullptr, nullptr, c->dz[l - 1]);
  }
  CCHK(c, hipGetLastError());
  CCHK(c, hipMemcpyAsync(c->lpart_h, c->lpart, 1024 * sizeof(double), hipMemcpyDeviceToHost,
                         c->stream));
  CCHK(c, hipStreamSynchronize(c->stream));
  double s = 0.0;
  for (int i = 0; i < 1024; ++i) s += c->lpart_h[i];
  if (loss) *loss = s / (double)nv;
  c->grad_valid = true;
  return HMC_OK;
}

}  // namespace

extern "C" {

size_t cnn_param_count(void) { return (size_t)n_params(); }

const char* cnn_last_error(const cnn_ctx* c) { return c ? c->err.c_str() : g_cerr.c_str(); }

void cnn_destroy(cnn_ctx* c) {
  if (!c) return;
  if (c->stream) (void)hipStreamSynchronize(c->stream);
  free_acts(c);
  (void)hipFree(c->p);
  (void)hipFree(c->g);
  (void)hipFree(c->m1);
  (void)hipFree(c->m2);
  for (int l = 0; l < 4; ++l) {
    (void)hipFree(c->wp[l]);
    (void)hipFree(c->wd[l]);
  }
  (void)hipFree(c->wpart);
  (void)hipFree(c->dbpart);
  (void)hipFree(c->lpart);
  if (c->lpart_h) (void)hipHostFree(c->lpart_h);
  delete c;
}

hmc_status cnn_create(const float* params, void* stream, cnn_ctx** out) {
  if (!out || !params) return cfail(nullptr, HMC_EINVAL, "null argument");
  cnn_ctx* c = new cnn_ctx();
  c->stream = (hipStream_t)stream;
  const int np = n_params();
  auto bail = [&](const char* what, hipError_t e) {
    c->err = std::string(what) + ": " + hipGetErrorString(e);
    g_cerr = c->err;
    cnn_destroy(c);
    return HMC_EDEVICE;
  };
  hipError_t e;
  // g holds the gradient and, past its end, the last layer's bias padded to 16
  if ((e = hipMalloc(&c->p, np * sizeof(float))) != hipSuccess) return bail("hipMalloc", e);
  if ((e = hipMalloc(&c->g, n_grad() * sizeof(float))) != hipSuccess) return bail("hipMalloc", e);
  if ((e = hipMalloc(&c->m1, np * sizeof(float))) != hipSuccess) return bail("hipMalloc", e);
  if ((e = hipMalloc(&c->m2, np * sizeof(float))) != hipSuccess) return bail("hipMalloc", e);
  for (int l = 0; l < 4; ++l) {
    if ((e = hipMalloc(&c->wp[l], nchunk_fwd(l) * 64 * sizeof(bf16x4))) != hipSuccess)
      return bail("hipMalloc", e);
    if ((e = hipMalloc(&c->wd[l], 27 * 64 * sizeof(bf16x4))) != hipSuccess) return bail("hipMalloc", e);
  }
  if ((e = hipMalloc(&c->wpart, (size_t)kParts * kTile * sizeof(float))) != hipSuccess)
    return bail("hipMalloc", e);
  if ((e = hipMalloc(&c->dbpart, (size_t)kParts * 16 * sizeof(float))) != hipSuccess)
    return bail("hipMalloc", e);
  if ((e = hipMalloc(&c->lpart, 1024 * sizeof(double))) != hipSuccess) return bail("hipMalloc", e);
  if ((e = hipHostMalloc((void**)&c->lpart_h, 1024 * sizeof(double), 0)) != hipSuccess)
    return bail("hipHostMalloc", e);
  std::vector<float> zeros(n_grad(), 0.f);
  if ((e = hipMemcpy(c->p, params, np * sizeof(float), hipMemcpyHostToDevice)) != hipSuccess)
    return bail("upload", e);
  if ((e = hipMemcpy(c->m1, zeros.data(), np * sizeof(float), hipMemcpyHostToDevice)) != hipSuccess ||
      (e = hipMemcpy(c->m2, zeros.data(), np * sizeof(float), hipMemcpyHostToDevice)) != hipSuccess ||
      (e = hipMemcpy(c->g, zeros.data(), n_grad() * sizeof(float), hipMemcpyHostToDevice)) != hipSuccess)
    return bail("upload", e);
  // padded last-layer bias after the gradient
  if ((e = hipMemcpy(c->g + off_pad(), params + off_b(3), 2 * sizeof(float), hipMemcpyHostToDevice)) != hipSuccess)
    return bail("upload", e);
  if (pack_all(c) != HMC_OK) {
    g_cerr = c->err;
    cnn_destroy(c);
    return HMC_EDEVICE;
  }
  *out = c;
  return HMC_OK;
}

hmc_status cnn_get_params(cnn_ctx* c, float* params) {
  if (!c || !params) return cfail(c, HMC_EINVAL, "null argument");
  CCHK(c, hipMemcpyAsync(params, c->p, n_params() * sizeof(float), hipMemcpyDeviceToHost, c->stream));
  CCHK(c, hipStreamSynchronize(c->stream));
  return HMC_OK;
}

hmc_status cnn_forward(cnn_ctx* c, int32_t n, const float* in3, float* mu, float* logvar) {
  if (!c || !in3) return cfail(c, HMC_EINVAL, "null argument");
  hmc_status st = ensure(c, n);
  if (st != HMC_OK) return st;
  return infer(c, n, in3, mu, logvar);
}

hmc_status cnn_features(cnn_ctx* c, int32_t n, const float* beta, float beta_scale,
                        const float* mask, const float* sel, float* out3) {
  if (!c || !beta || !mask || !sel || !out3 || n < 4) return cfail(c, HMC_EINVAL, "bad argument");
  const long long nv = (long long)n * n * n;
  hipLaunchKernelGGL(k_features, dim3(4096), dim3(256), 0, c->stream, nv, beta, beta_scale, mask,
                     sel, out3);
  CCHK(c, hipGetLastError());
  return HMC_OK;
}

hmc_status cnn_gradient(cnn_ctx* c, int32_t n, const float* in3, const float* target, float* grad,
                        double* loss) {
  if (!c || !in3 || !target) return cfail(c, HMC_EINVAL, "null argument");
  hmc_status st = ensure(c, n);
  if (st != HMC_OK) return st;
  if ((st = gradient(c, n, in3, target, loss)) != HMC_OK) return st;
  if (grad) {
    CCHK(c, hipMemcpyAsync(grad, c->g, n_params() * sizeof(float), hipMemcpyDeviceToHost, c->stream));
    CCHK(c, hipStreamSynchronize(c->stream));
  }
  return HMC_OK;
}

hmc_status cnn_layer_state(cnn_ctx* c, int32_t layer, float* z, float* a, float* dz) {
  if (!c || layer < 0 || layer > 3 || (layer == 3 && a)) return cfail(c, HMC_EINVAL, "bad argument");
  if (c->n == 0 || !c->grad_valid) return cfail(c, HMC_EINVAL, "no cnn_gradient or cnn_train_step yet");
  const long long nv = (long long)c->n * c->n * c->n;
  hipLaunchKernelGGL(k_layer_state, dim3(4096), dim3(256), 0, c->stream, nv, kCout[layer],
                     layer < 3 ? 16 : 2, c->z[layer], layer < 3 ? c->a[layer] : nullptr, c->dz[layer], z, a, dz);
  CCHK(c, hipGetLastError());
  return HMC_OK;
}

hmc_status cnn_gelu_check(cnn_ctx* c, uint32_t first, uint64_t count, uint32_t seed, int64_t* differ,
                          double* worst) {
  if (!c || !differ || !worst || count == 0 || count % 4 != 0 || first + count > (1ull << 32))
    return cfail(c, HMC_EINVAL, "bad argument");
  // lpart holds nothing between calls
  for (int i = 0; i < 3; ++i) c->lpart_h[i] = 0.0;
  CCHK(c, hipMemcpyAsync(c->lpart, c->lpart_h, 3 * sizeof(double), hipMemcpyHostToDevice, c->stream));
  hipLaunchKernelGGL(k_gelu_check, dim3(2048), dim3(256), 0, c->stream, first, (uint32_t)(count / 4), seed,
                     (unsigned long long*)c->lpart);
  CCHK(c, hipGetLastError());
  CCHK(c, hipMemcpyAsync(c->lpart_h, c->lpart, 3 * sizeof(double), hipMemcpyDeviceToHost, c->stream));
  CCHK(c, hipStreamSynchronize(c->stream));
  memcpy(differ, c->lpart_h, 2 * sizeof(int64_t));
  float w[2];
  memcpy(w, c->lpart_h + 2, sizeof(w));
  worst[0] = w[0];
  worst[1] = w[1];
  return HMC_OK;
}

hmc_status cnn_train_step(cnn_ctx* c, int32_t n, const float* in3, const float* target, float lr,
                          double* loss) {
  if (!c || !in3 || !target || !(lr > 0)) return cfail(c, HMC_EINVAL, "bad argument");
  hmc_status st = ensure(c, n);
  if (st != HMC_OK) return st;
  if ((st = gradient(c, n, in3, target, loss)) != HMC_OK) return st;
  c->steps += 1;
  const float c1 = 1.f - std::pow(0.9f, (float)c->steps), c2 = 1.f - std::pow(0.999f, (float)c->steps);
  const int np = n_params();
  hipLaunchKernelGGL(k_adam, dim3((np + 255) / 256), dim3(256), 0, c->stream, np, c->p, c->g, c->m1,
                     c->m2, lr, c1, c2);
  // keep the padded last-layer bias in step with the master copy
  CCHK(c, hipMemcpyAsync(c->g + off_pad(), c->p + off_b(3), 2 * sizeof(float), hipMemcpyDeviceToDevice,
                         c->stream));
  return pack_all(c);
}

}  // extern "C"
