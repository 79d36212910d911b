// Learned shrinkage network on gfx950 matrix cores (an extension beyond the
// paper: a per-scale CNN predicting a gain in [0, 1] for every detail
// coefficient; hard thresholding, Section 5.3, is its fallback).
//
//   x0 = (|c| / (sigma ||psi_i||_2), sigma * 255 / 50)        2 channels
//   h1 = relu(conv3x3(x0; W1) + b1)     h2 = relu(conv3x3(h1; W2) + b2)
//   g  = sigmoid(conv3x3(h2; W3) + b3)  shrunk coefficient g * c
//
// Activations are channel-last bfloat16 tensors [P][H][W][32] (P planes, 64 B
// per pixel, unused channels zero).  A 3x3 convolution is an implicit GEMM:
// for every tap, 16 output pixels x 16 output channels accumulate one
// v_mfma_f32_16x16x32_bf16 over the 32 input channels (FP32 accumulation).
// Operand layout of that instruction (64 lanes, l = lane):
//   A[m][k]: m = l % 16, k = 8 (l / 16) + j, j = 0..7  (8 bf16 per lane)
//   B[k][n]: n = l % 16, k = 8 (l / 16) + j
//   D[m][n]: n = l % 16, m = 4 (l / 16) + i, i = 0..3  (4 floats per lane)
// The backward pass is in cnn_bwd.hip.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "cnn.hpp"
#include "cnn_device.hpp"

namespace sl {

constexpr int TH = 8, TW = 32;                 // output tile
constexpr int HH = TH + 2, HW2 = TW + 2;       // input halo tile

// ---------------------------------------------------------------------------
// x0 planes from the coefficients
// ---------------------------------------------------------------------------
__global__ void k_cnn_x0(const float *__restrict__ coef, CnnPlanes pl, uint16_t *__restrict__ x0,
                         int HWn) {
  const int p = blockIdx.y;
  const int px = blockIdx.x * blockDim.x + threadIdx.x;
  if (px >= HWn) return;
  int b, i, j;
  plane_info(pl, p, b, i, j);
  const float sg = pl.sigma[b];
  const float c = coef[((size_t)b * pl.R + i) * HWn + px];
  const float v0 = fabsf(c) / (sg * pl.l2[i]);
  const float v1 = sg * (255.0f / 50.0f);
  uint4 *dst = (uint4 *)(x0 + ((size_t)p * HWn + px) * CH);
  dst[0] = make_uint4((uint32_t)f2bf(v0) | ((uint32_t)f2bf(v1) << 16), 0u, 0u, 0u);
  dst[1] = make_uint4(0u, 0u, 0u, 0u);
  dst[2] = make_uint4(0u, 0u, 0u, 0u);
  dst[3] = make_uint4(0u, 0u, 0u, 0u);
}

// ---------------------------------------------------------------------------
// 3x3 convolution, implicit GEMM on MFMA
// ---------------------------------------------------------------------------
// Wp: packed weight operands [J][9][NB][64 lanes][8] bf16; bias [J][..] float.
// The weights are the A operand and the activation tile the B operand, so a
// lane receives 4 consecutive output channels (16 nb + 4 (lane / 16) + i) of
// one pixel (lane % 16) and stores them with one 8-byte write.  The halo tile
// keeps pixels at a 40-channel stride (80 bytes) in LDS.
constexpr int kConvCP = 40;
template <int NB, int MODE>
__global__ void __launch_bounds__(256)
k_conv3x3(const uint16_t *__restrict__ in, const uint16_t *__restrict__ Wp,
          const float *__restrict__ bias, int bias_stride, CnnPlanes pl, int H, int W,
          uint16_t *__restrict__ out, const float *__restrict__ coef, float *__restrict__ coef_out,
          float *__restrict__ gain) {
  __shared__ __attribute__((aligned(16))) uint16_t tile[HH * HW2 * kConvCP];
  const int p = blockIdx.z;
  const int ty0 = blockIdx.y * TH, tx0 = blockIdx.x * TW;
  const size_t HWn = (size_t)H * W;
  const uint16_t *src = in + (size_t)p * HWn * CH;
  int b, i, j;
  plane_info(pl, p, b, i, j);
  // halo tile: 16-byte chunks, zero outside the image
  for (int q = threadIdx.x; q < HH * HW2 * 4; q += 256) {
    const int pix = q >> 2, part = q & 3;
    const int yy = ty0 + pix / HW2 - 1, xx = tx0 + pix % HW2 - 1;
    uint4 v = make_uint4(0u, 0u, 0u, 0u);
    if (yy >= 0 && yy < H && xx >= 0 && xx < W)
      v = ((const uint4 *)(src + ((size_t)yy * W + xx) * CH))[part];
    *(uint4 *)(tile + pix * kConvCP + 8 * part) = v;
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g = lane >> 4;
  bf16x8 wb[9][NB];
  const uint16_t *wj = Wp + (size_t)j * 9 * NB * 64 * 8;
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
      wb[t][nb] = *(const bf16x8 *)(wj + (((size_t)t * NB + nb) * 64 + lane) * 8);
  // accumulator initial values: the bias of each lane's 4 channels (layer 3
  // has one output channel, channel 0)
  f32x4 binit[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int ch = 16 * nb + 4 * g + e;
      float v = 0.f;
      if constexpr (MODE == CONV_RELU) v = bias[(size_t)j * bias_stride + ch];
      if constexpr (MODE == CONV_GAIN) v = ch == 0 ? bias[(size_t)j * bias_stride] : 0.f;
      binit[nb][e] = v;
    }
  __syncthreads();
  // 16 pixel blocks (row r, half h) per tile; wave w takes blocks w, w+4, w+8, w+12
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const int blk = wave + 4 * s;
    const int r = blk >> 1, c0 = (blk & 1) * 16;
    f32x4 acc[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[nb] = binit[nb];
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      const int dy = t / 3, dx = t % 3;
      const int pix = (r + dy) * HW2 + c0 + (lane & 15) + dx;
      const bf16x8 xb = *(const bf16x8 *)(tile + pix * kConvCP + 8 * g);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
        acc[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wb[t][nb], xb, acc[nb], 0, 0, 0);
    }
    const int yy = ty0 + r, xx = tx0 + c0 + (lane & 15);
    if (yy >= H || xx >= W) continue;
    const size_t opix = (size_t)p * HWn + (size_t)yy * W + xx;
    if constexpr (MODE == CONV_RELU) {
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        bf16x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = (__bf16)fmaxf(acc[nb][e], 0.f);
        *(bf16x4 *)(out + opix * CH + 16 * nb + 4 * g) = o;
      }
    } else {   // CONV_GAIN: channel 0 sits in lane group 0, element 0
      if (g == 0) {
        const float gv = 1.0f / (1.0f + __expf(-acc[0][0]));
        const size_t co = ((size_t)b * pl.R + i) * HWn + (size_t)yy * W + xx;
        if (gain) gain[co] = gv;
        if (coef_out) coef_out[co] = gv * coef[co];
      }
    }
  }
}

// ---------------------------------------------------------------------------
// fused inference: the three layers of 12 x 32 output tiles in LDS
// ---------------------------------------------------------------------------
// Regions (rows x cols): x0 18 x 38, h1 16 x 36, h2 14 x 34, output 12 x 32.
// Activations outside the image are zero (the "same" zero padding of every
// layer).  Layer 1 packs its 9 taps x 2 input channels into one K = 32
// operand (k = 2 t + c, k >= 18 zero); layer 2 is the per-tap implicit GEMM.
// Layer 3 has one output channel: a product with the 9 taps on the M axis
// yields D[t][p] = sum_ci W3[ci][t] h2[p][ci], and the output is
// b3 + sum_t D[t][p + offset(t)]; h2 never reaches LDS.
//
// A wave computes 16 of the 32 channels of layer 2 (nb = wave % 2), so its
// operands take 36 registers instead of 72 and two blocks of 8 waves run per
// compute unit (128 registers, 74 KiB of LDS): one block's matrix products
// overlap the other's element work and barriers.  Layer 2 streams down two
// 16-pixel strips (three shifted operands of an input row feed three output
// rows, a third of the LDS reads of nine operands per row); the two columns
// left over go in two blocks.  Each half of the channels leaves its own layer-3
// sums D in LDS (adding them there with LDS atomics took 13 ms per 8 images);
// 12 rows keep both within two blocks' share.
// One 512-thread block per CU holding all 72 operand registers per wave, nine
// LDS operands per 16 pixels and 48-channel pixel strides: 16.4 ms per
// 32 x 512^2 images; this form 12.9 ms (8 images denoised with the
// network: 4713 -> 3723 us).
constexpr int FTH = 12, FTW = 32;
constexpr int X0H = FTH + 6, X0W = FTW + 6;
constexpr int H1H = FTH + 4, H1W = FTW + 4;
constexpr int H2H = FTH + 2, H2W = FTW + 2;
constexpr int NX0 = X0H * X0W, NH1 = H1H * H1W, NH2 = H2H * H2W;
constexpr int kFusedThreads = 512, kFusedWaves = kFusedThreads / 64;
static_assert(NH1 % 16 == 0 && H2W == 34, "tile geometry");
constexpr int kX0PerThread = (NX0 + kFusedThreads - 1) / kFusedThreads;
// LDS (bytes): h1 | layer-3 sums D[2][9][NH2] | x0
constexpr int kFOD3 = NH1 * kPix, kFOX0 = kFOD3 + 2 * 9 * NH2 * 4, kLdsFused = kFOX0 + NX0 * 4;
constexpr int kFusedBlocksPerCU = 2;
static_assert(kFusedBlocksPerCU * kLdsFused <= 160 * 1024, "LDS of a compute unit");

struct FusedTile {
  int p, ty0, tx0, b, i, j;
};

__device__ __forceinline__ FusedTile fused_tile(const CnnPlanes &pl, int tile, int tiles_x,
                                                int tiles_per_plane) {
  FusedTile f;
  f.p = tile / tiles_per_plane;
  const int r = tile % tiles_per_plane;
  f.ty0 = (r / tiles_x) * FTH;
  f.tx0 = (r % tiles_x) * FTW;
  plane_info(pl, f.p, f.b, f.i, f.j);
  return f;
}

__global__ void __launch_bounds__(kFusedThreads, 4)
k_cnn_fused(const float *__restrict__ coef, CnnPlanes pl, int H, int W, int ntiles,
            const uint16_t *__restrict__ W1k, const uint16_t *__restrict__ W2p,
            const uint16_t *__restrict__ W3p, const float *__restrict__ params,
            float *__restrict__ coef_out, float *__restrict__ gain) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[kLdsFused];
  float *d3 = (float *)(smem + kFOD3);
  uint32_t *x0s = (uint32_t *)(smem + kFOX0);
  const int lane = threadIdx.x & 63, n0 = lane & 15, g0 = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nb = wave & 1, strip = (wave >> 1) & 1, half = wave >> 2;
  const int tiles_x = (W + FTW - 1) / FTW;
  const int tiles_per_plane = tiles_x * ((H + FTH - 1) / FTH);
  const size_t HWn = (size_t)H * W;

  // coefficients of the x0 region and of the thread's output pixel
  float xr[kX0PerThread], cen;
  auto fetch = [&](const FusedTile &f) {
    const float *cpl = coef + ((size_t)f.b * pl.R + f.i) * HWn;
    const int tid = fresh(threadIdx.x);
#pragma unroll
    for (int u = 0; u < kX0PerThread; ++u) {
      const int q = tid + u * kFusedThreads, r = (q * 1725) >> 16;       // q / 38
      const int yy = f.ty0 - 3 + r, xx = f.tx0 - 3 + q - r * X0W;
      const bool in = q < NX0 && (unsigned)yy < (unsigned)H && (unsigned)xx < (unsigned)W;
      xr[u] = in ? cpl[yy * W + xx] : 0.f;
    }
    const int yy = f.ty0 + (tid >> 5), xx = f.tx0 + (tid & 31);
    cen = (tid < FTH * FTW && yy < H && xx < W) ? cpl[yy * W + xx] : 0.f;
  };
  auto stage = [&](const FusedTile &f) {
    const float sg = pl.sigma[f.b];
    const float inv = 1.0f / (sg * pl.l2[f.i]);
    const uint32_t ch1 = (uint32_t)f2bf(sg * (255.0f / 50.0f)) << 16;
    const int tid = fresh(threadIdx.x);
#pragma unroll
    for (int u = 0; u < kX0PerThread; ++u) {
      const int q = tid + u * kFusedThreads, r = (q * 1725) >> 16;
      // out-of-image positions were fetched as 0; their x0 must be 0 in both channels
      const int yy = f.ty0 - 3 + r, xx = f.tx0 - 3 + q - r * X0W;
      const bool in = (unsigned)yy < (unsigned)H && (unsigned)xx < (unsigned)W;
      if (q < NX0) x0s[q] = in ? ((uint32_t)f2bf(fabsf(xr[u]) * inv) | ch1) : 0u;
    }
  };

  // operands of the current scale (reloaded when the scale changes); the
  // biases are the accumulators' initial values
  bf16x8 w1[2], w2[9];
  s16x4 w3;
  f32x4 bias1[2], bias2;
  float b3 = 0.f;
  auto load_weights = [&](int j) {
    const float *P = params + (size_t)j * kCnnParams;
    // layer 3, taps on M, this wave's 16 channels on K: row n, k = 4 g + e (four
    // channels of a tap lie together in the pack)
    const int tap = fresh(n0);
    const s16x4 w3p = *(const s16x4 *)packed_w3(W3p, j, 16 * nb + 4 * fresh(g0), min(tap, 8));
#pragma unroll
    for (int e = 0; e < 4; ++e) w3[e] = tap < 9 ? w3p[e] : (short)0;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      w1[b] = *(const bf16x8 *)(W1k + (((size_t)j * 2 + b) * 64 + lane) * 8);
#pragma unroll
      for (int e = 0; e < 4; ++e) bias1[b][e] = P[kOffB1 + 16 * b + 4 * g0 + e];
    }
#pragma unroll
    for (int t = 0; t < 9; ++t)
      w2[t] = *(const bf16x8 *)(W2p + ((((size_t)j * 9 + t) * 2 + nb) * 64 + lane) * 8);
#pragma unroll
    for (int e = 0; e < 4; ++e) bias2[e] = P[kOffB2 + 16 * nb + 4 * g0 + e];
    b3 = P[kOffB3];
  };
  // relu and layer 3 of 16 pixels at d3 index q of lane n
  auto layer3 = [&](f32x4 a, uint32_t in, int q, int g) {
    const uint2 h = relu_pack(a, in);
    const f32x4 d = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(w3, *(const s16x4 *)&h,
                                                              f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
    float *dp = d3 + (9 * nb + 4 * g) * NH2 + q;
    if (g < 3) dp[0] = d[0];
    if (g < 2) {
#pragma unroll
      for (int e = 1; e < 4; ++e) dp[e * NH2] = d[e];
    }
  };

  int tile = blockIdx.x;
  if (tile >= ntiles) return;
  int cur_j = -1;
  FusedTile f = fused_tile(pl, tile, tiles_x, tiles_per_plane);
  fetch(f);
  stage(f);
  float cc = cen;
  for (;;) {
    if (f.j != cur_j) {
      load_weights(f.j);
      cur_j = f.j;
    }
    const bool interior = f.ty0 >= 3 && f.ty0 + FTH + 3 <= H && f.tx0 >= 3 && f.tx0 + FTW + 3 <= W;
    __syncthreads();
    // ---- layer 1 (36 blocks of 16 pixels, three and two at a time; waves
    // without a fifth block repeat block 35) ----
    {
      const int n = fresh(n0), g = fresh(g0);
      // dword h of a lane's K slice is the (channel 0, channel 1) pair of tap
      // 4 g + h; the slots of taps >= 9 have zero weights and read tap 0
      int toff[4];
#pragma unroll
      for (int h = 0; h < 4; ++h) {
        const int t = 4 * g + h, dy = (t * 11) >> 5;               // t / 3
        toff[h] = t < 9 ? dy * X0W + t - 3 * dy : 0;
      }
      auto l1 = [&](int b0, auto count) {
        constexpr int S = decltype(count)::value;
        bf16x8 xb[S];
        int o[S];
        uint32_t in[S];
#pragma unroll
        for (int s = 0; s < S; ++s) {
          const int q = min(b0 + kFusedWaves * s, NH1 / 16 - 1) * 16 + n;
          const int r = (q * 1821) >> 16, c = q - r * H1W;         // q / 36
          const int base = q + 2 * r;                              // r X0W + c
          uint32_t u[4];
#pragma unroll
          for (int h = 0; h < 4; ++h) u[h] = x0s[base + toff[h]];
          xb[s] = *(const bf16x8 *)u;
          o[s] = q * kPix + (swz(c, g >> 1) | (g & 1) * 8);
          in[s] = 0xFFFFFFFFu;
          if (!interior) {
            const int yy = f.ty0 - 2 + r, xx = f.tx0 - 2 + c;
            in[s] = ((unsigned)yy < (unsigned)H && (unsigned)xx < (unsigned)W) ? 0xFFFFFFFFu : 0u;
          }
        }
        f32x4 d[S][2];
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
          for (int b = 0; b < 2; ++b) d[s][b] = mma(w1[b], xb[s], bias1[b]);
#pragma unroll
        for (int s = 0; s < S; ++s) {
          *(uint2 *)(smem + o[s]) = relu_pack(d[s][0], in[s]);
          *(uint2 *)(smem + (o[s] ^ 32)) = relu_pack(d[s][1], in[s]);
        }
      };
      static_assert((NH1 / 16 + kFusedWaves - 1) / kFusedWaves == 5, "layer-1 blocks per wave");
      l1(wave, IntC<3>{});
      l1(wave + 3 * kFusedWaves, IntC<2>{});
    }
    // the next tile's coefficients land during layer 2
    const int next = tile + gridDim.x;
    FusedTile fn = f;
    if (next < ntiles) {
      fn = fused_tile(pl, next, tiles_x, tiles_per_plane);
      fetch(fn);
    }
    __syncthreads();
    // ---- layers 2 and 3: columns 0..31 in two strips of two halves of 7
    // rows; columns 32, 33 in two blocks of 16 (8 rows) ----
    {
      constexpr int RH = H2H / 2;
      const int n = fresh(n0), g = fresh(g0);
      const int r0 = RH * half, c = 16 * strip + n;
      int ad[3];
#pragma unroll
      for (int dx = 0; dx < 3; ++dx) ad[dx] = (r0 * H1W + c + dx) * kPix + swz(c + dx, g);
      const bool cin = (unsigned)(f.tx0 - 1 + c) < (unsigned)W;
      f32x4 acc[3];
      bf16x8 fr[2][3];
#pragma unroll
      for (int dx = 0; dx < 3; ++dx) fr[0][dx] = *(const bf16x8 *)(smem + ad[dx]);
#pragma unroll
      for (int y = 0; y < RH + 2; ++y) {
        if (y + 1 < RH + 2) {
#pragma unroll
          for (int dx = 0; dx < 3; ++dx)
            fr[(y + 1) & 1][dx] = *(const bf16x8 *)(smem + ad[dx] + (y + 1) * H1W * kPix);
        }
        if (y < RH) acc[y % 3] = bias2;
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int dx = 0; dx < 3; ++dx)
#pragma unroll
          for (int dy = 2; dy >= 0; --dy) {
            const int r = y - dy;
            if (r >= 0 && r < RH) acc[r % 3] = mma(w2[3 * dy + dx], fr[y & 1][dx], acc[r % 3]);
          }
        __builtin_amdgcn_s_setprio(0);
        if (y >= 2) {
          const int yy = f.ty0 - 1 + r0 + y - 2;
          const uint32_t in = (cin && (unsigned)yy < (unsigned)H) ? 0xFFFFFFFFu : 0u;
          layer3(acc[(y - 2) % 3], in, (r0 + y - 2) * H2W + c, g);
        }
      }
      if (wave < 4) {
        const int lc = min((wave >> 1) * 16 + n, 2 * H2H - 1);
        const int r = lc >> 1, cl = 32 + (lc & 1);
        f32x4 a = bias2;
        int o[3];
#pragma unroll
        for (int dx = 0; dx < 3; ++dx) o[dx] = (r * H1W + cl + dx) * kPix + swz(cl + dx, g);
#pragma unroll
        for (int k = 0; k < 9; ++k)
          a = mma(w2[k], *(const bf16x8 *)(smem + o[k % 3] + (k / 3) * H1W * kPix), a);
        const int yy = f.ty0 - 1 + r, xx = f.tx0 - 1 + cl;
        const uint32_t in = ((unsigned)yy < (unsigned)H && (unsigned)xx < (unsigned)W) ? 0xFFFFFFFFu : 0u;
        // (lanes past the last pixel repeat it)
        layer3(a, in, r * H2W + cl, g);
      }
    }
    __syncthreads();
    // ---- output: one pixel per thread; then the next tile's x0 ----
    {
      const int tid = fresh(threadIdx.x), r = tid >> 5, c = tid & 31;
      const int yy = f.ty0 + r, xx = f.tx0 + c;
      if (r < FTH && yy < H && xx < W) {
        float z = b3;
#pragma unroll
        for (int t = 0; t < 9; ++t) {
          const float *dp = d3 + t * NH2 + (r + t / 3) * H2W + c + t % 3;
          z += dp[0] + dp[9 * NH2];
        }
        const float gv = 1.0f / (1.0f + __expf(-z));
        const size_t co = ((size_t)f.b * pl.R + f.i) * HWn + (size_t)yy * W + xx;
        if (gain) gain[co] = gv;
        coef_out[co] = gv * cc;
      }
    }
    if (next >= ntiles) break;
    stage(fn);
    cc = cen;
    tile = next;
    f = fn;
  }
}

// Sum of n block partials in a fixed order: one block, a strided sum per
// thread, then a tree (one thread walking 1024 partials took 65 us).
__global__ void __launch_bounds__(256)
k_sum_partials(const float *__restrict__ partial, int n, float *__restrict__ outv) {
  __shared__ float red[256];
  float s = 0.f;
  for (int q = threadIdx.x; q < n; q += 256) s += partial[q];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) outv[0] = red[0];
}

// Pack the conv B operands of every scale from the FP32 parameter blobs,
// layout [J][taps][NB][64 lanes][8]:
// mode 0: forward layer (W[co][ci][t]); mode 1: transposed layer with flipped
// taps (W'[ci][co][8 - t]) for the backward data pass; mode 2: layer 1 with
// its 9 taps x 2 channels packed into one K = 32 operand (taps = 1).
__global__ void k_pack(const float *__restrict__ params, int J, int layer, int mode,
                       uint16_t *__restrict__ Wp, int NB) {
  const int taps = mode == 2 ? 1 : 9;
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;   // over J*taps*NB*64*8
  const int total = J * taps * NB * 64 * 8;
  if (idx >= total) return;
  const int jj = idx % 8, lane = (idx / 8) % 64, nb = (idx / 512) % NB;
  const int t = (idx / (512 * NB)) % taps;
  const int js = idx / (512 * NB * taps);
  const int n = 16 * nb + (lane & 15);          // output channel of this conv
  const int k = 8 * (lane >> 4) + jj;           // input channel of this conv
  const float *P = params + (size_t)js * kCnnParams;
  float v = 0.f;
  // forward weight of the requested layer: Wl[co][ci][t] with sizes (cout, cin)
  const int off[3] = {kOffW1, kOffW2, kOffW3};
  const int cin[3] = {2, 32, 32}, cout[3] = {32, 32, 1};
  const int l = layer - 1;
  if (mode == 2) {
    const int tt = k >> 1, cc = k & 1;
    if (n < 32 && tt < 9) v = P[off[0] + (n * 2 + cc) * 9 + tt];
  } else if (mode == 0) {
    if (n < cout[l] && k < cin[l]) v = P[off[l] + (n * cin[l] + k) * 9 + t];
  } else {
    // transposed: this conv maps the layer's output channels (k) to its input channels (n)
    if (n < cin[l] && k < cout[l]) v = P[off[l] + (k * cin[l] + n) * 9 + (8 - t)];
  }
  Wp[idx] = f2bf(v);
}

// Adam (Kingma and Ba) on the FP32 master parameters.  The constants b1,
// 1 - b1, b2, 1 - b2 and the bias corrections c1 = 1 - b1^t, c2 = 1 - b2^t
// are formed in double on the host and rounded once (1 - 0.999f in float32
// would be 1.3e-5 off 0.001).
__global__ void k_adam(float *__restrict__ p, const float *__restrict__ g, float *__restrict__ m,
                       float *__restrict__ v, int n, float lr, float b1, float omb1, float b2,
                       float omb2, float eps, float c1, float c2) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const float gg = g[k];
  const float mm = b1 * m[k] + omb1 * gg;
  const float vv = b2 * v[k] + omb2 * gg * gg;
  m[k] = mm;
  v[k] = vv;
  p[k] -= lr * (mm / c1) / (sqrtf(vv / c2) + eps);
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
hipError_t cnn_x0(const float *coef, const CnnPlanes &pl, int P, int H, int W, uint16_t *x0,
                  hipStream_t st) {
  const int HWn = H * W;
  hipLaunchKernelGGL(k_cnn_x0, dim3((HWn + 255) / 256, P), dim3(256), 0, st, coef, pl, x0, HWn);
  return hipGetLastError();
}

hipError_t cnn_conv(const uint16_t *in, const uint16_t *Wp, int NB, const float *bias,
                    int bias_stride, const CnnPlanes &pl, int P, int H, int W, int mode,
                    uint16_t *out, const float *coef, float *coef_out, float *gain,
                    hipStream_t st) {
  dim3 grid((W + TW - 1) / TW, (H + TH - 1) / TH, P);
  if (mode == CONV_RELU && NB == 2)
    hipLaunchKernelGGL((k_conv3x3<2, CONV_RELU>), grid, dim3(256), 0, st, in, Wp, bias,
                       bias_stride, pl, H, W, out, coef, coef_out, gain);
  else if (mode == CONV_GAIN && NB == 1)
    hipLaunchKernelGGL((k_conv3x3<1, CONV_GAIN>), grid, dim3(256), 0, st, in, Wp, bias,
                       bias_stride, pl, H, W, out, coef, coef_out, gain);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t cnn_fused(const float *coef, const CnnPlanes &pl, int P, int H, int W,
                     const uint16_t *W1k, const uint16_t *W2p, const uint16_t *W3p,
                     const float *params, float *coef_out, float *gain, int nblocks,
                     hipStream_t st) {
  const int ntiles = P * ((W + FTW - 1) / FTW) * ((H + FTH - 1) / FTH);
  nblocks *= kFusedBlocksPerCU;
  const int grid = nblocks < ntiles ? nblocks : ntiles;
  if (grid < 1) return hipSuccess;
  hipLaunchKernelGGL(k_cnn_fused, dim3(grid), dim3(kFusedThreads), 0, st, coef, pl, H, W, ntiles,
                     W1k, W2p, W3p, params, coef_out, gain);
  return hipGetLastError();
}

__global__ void k_copy_lowpass(const float *__restrict__ coef, float *__restrict__ out, int R,
                               int HWn) {
  const int b = blockIdx.y;
  const int px = blockIdx.x * blockDim.x + threadIdx.x;
  if (px < HWn) out[(size_t)b * R * HWn + px] = coef[(size_t)b * R * HWn + px];
}

// out = scale (a - b); partial[block] = sum of (a - b)^2 over the block's stride
__global__ void k_sqerr(const float *__restrict__ a, const float *__restrict__ b, size_t n,
                        float scale, float *__restrict__ out, float *__restrict__ partial) {
  __shared__ float red[256];
  float s = 0.f;
  for (size_t k = (size_t)blockIdx.x * 256 + threadIdx.x; k < n; k += (size_t)gridDim.x * 256) {
    const float d = a[k] - b[k];
    out[k] = scale * d;
    s += d * d;
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

hipError_t sq_error_grad(const float *a, const float *b, size_t n, float scale, float *out,
                         float *partial, int nblocks, float *loss, hipStream_t st) {
  hipLaunchKernelGGL(k_sqerr, dim3(nblocks), dim3(256), 0, st, a, b, n, scale, out, partial);
  hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(256), 0, st, partial, nblocks, loss);
  return hipGetLastError();
}

hipError_t cnn_copy_lowpass(const float *coef, float *coef_out, int B, int R, int HWn,
                            hipStream_t st) {
  hipLaunchKernelGGL(k_copy_lowpass, dim3((HWn + 255) / 256, B), dim3(256), 0, st, coef, coef_out,
                     R, HWn);
  return hipGetLastError();
}

hipError_t cnn_pack(const float *params, int J, int layer, int mode, uint16_t *Wp, int NB,
                    hipStream_t st) {
  // mode 2 (packed layer 1) has one operand per (scale, nb): index as taps = 1
  const int total = J * (mode == 2 ? 1 : 9) * NB * 64 * 8;
  hipLaunchKernelGGL(k_pack, dim3((total + 255) / 256), dim3(256), 0, st, params, J, layer, mode,
                     Wp, NB);
  return hipGetLastError();
}

hipError_t cnn_adam(float *p, const float *g, float *m, float *v, int n, float lr, double b1,
                    double b2, double eps, int t, hipStream_t st) {
  const float c1 = (float)(1.0 - std::pow(b1, (double)t));
  const float c2 = (float)(1.0 - std::pow(b2, (double)t));
  hipLaunchKernelGGL(k_adam, dim3((n + 255) / 256), dim3(256), 0, st, p, g, m, v, n, lr, (float)b1,
                     (float)(1.0 - b1), (float)b2, (float)(1.0 - b2), (float)eps, c1, c2);
  return hipGetLastError();
}

}  // namespace sl
