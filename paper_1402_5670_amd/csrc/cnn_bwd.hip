// Backward pass of the learned shrinkage network on gfx950 matrix cores: one
// kernel per call from coefficients and dL/d(shrunk coefficients) to the
// weight gradients of every scale, then a fixed-order sum of the blocks'
// partial gradients.
//
// A persistent block owns one scale and walks 16 x 32 tiles of its planes.
// Per tile it recomputes the forward activations and runs the backward
// chain in LDS; only the two coefficient tensors are read from memory (the
// layer-by-layer form moved 32-channel bfloat16 tensors of 64 bytes per
// coefficient through HBM fifteen times).  Regions around the owned tile T:
//   x0 on T+5 -> h1 on T+4 -> h2 on T+3 -> z, g, dz on T+2 -> da2 on T+1
//   -> da1 on T, and
//   dW3[t][ci] = sum_q h2[q][ci] dz[q - o(t)],     q in T
//   dW2[t][ci][co] = sum_p h1[p + o(t)][ci] da2[p][co],   p in T
//   dW1[t][c][co] = sum_p x0[p + o(t)][c] da1[p][co],     p in T
// with o(t) the tap offset; activations and gradients outside the image are
// zero, so every (pixel, tap) term is counted by exactly one tile.
//
// v_mfma_f32_16x16x32_bf16 (64 lanes, n = lane % 16, g = lane / 16):
//   A[m][k]: m = n, k = 8 g + j;  B[k][n]: k = 8 g + j;  D[m][n]: m = 4 g + e.
// Activations are pixel-major in LDS (cnn_device.hpp).  Convolutions read
// 8 channels of one pixel per lane; the weight gradients, whose reduction
// axis is the pixels, read 4 pixels of one channel per lane with the
// transposing LDS read (ds_read_b64_tr_b16).  Their 32 K slots are two
// vertically adjacent 16-pixel blocks: slot 8 g + j is pixel 4 g + j % 4 of
// row j / 4.
//
// Wave w: nb = w % 2 selects 16 output channels, so that each wave holds the
// operands of its half of W2 and of the transposed W2 in registers for the
// whole kernel (72 registers); with the weight gradients' accumulators that
// leaves two waves per SIMD.  The 3x3 convolutions stream down 16-pixel
// strips: an input row's three shifted operands feed three output rows, a
// third of the LDS reads of a convolution that reads nine operands per row.
//
// 4 x 512^2 images, 48 subbands each: one training step 34.5 ms with the
// layer-by-layer passes (about 30 of it backward), 6.5 ms with this kernel
// (4.5 ms; 29 thousand cycles a tile, 10 thousand of them matrix products: the
// rest is the LDS traffic of the operands, the element work and the barriers
// between the chain's steps).  One block of 8 waves per CU; 161 KB of LDS.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "cnn.hpp"
#include "cnn_device.hpp"

namespace sl {

namespace {

typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

constexpr int BH = 16, BW = 32;                    // owned tile
constexpr int XH = BH + 10, XW = BW + 10;          // x0
constexpr int AH = BH + 8, AW = BW + 8;            // h1
constexpr int EH = BH + 6, EW = BW + 6;            // h2
constexpr int ZH = BH + 4, ZW = BW + 4;            // dz
constexpr int DH = BH + 2, DW = BW + 2;            // da2
constexpr int kOH1 = 0;
constexpr int kOH2 = kOH1 + AH * AW * kPix;
constexpr int kODA = kOH2 + EH * EW * kPix;        // da2; before it, layer-3 partial sums
constexpr int kOX0 = kODA + DH * DW * kPix;
constexpr int kODZ = kOX0 + XH * XW * 4;
constexpr int kOZero = kODZ + ZH * ZW * 4;         // four zero words
constexpr int kLdsBwd = kOZero + 16;
constexpr int NE = EH * EW;                        // pixels of the h2 region
static_assert(9 * NE * 4 <= DH * DW * kPix, "layer-3 partial sums share the da2 region");
static_assert(kLdsBwd <= 160 * 1024, "LDS of a compute unit");
static_assert(kCnnParams * 4 <= AH * AW * kPix, "the final sum uses the h1 region");
constexpr int kBwdThreads = 512, NWV = kBwdThreads / 64;
constexpr int kXPer = (XH * XW + kBwdThreads - 1) / kBwdThreads;
constexpr int kZPer = (ZH * ZW + kBwdThreads - 1) / kBwdThreads;

// 16-bit halves of v kept where the halves of h (bfloat16) are not zero
__device__ __forceinline__ uint32_t keep_nonzero(uint32_t v, uint32_t h) {
  const uint32_t m = ((h & 0x7FFF7FFFu) + 0x7FFF7FFFu) & 0x80008000u;
  return v & ((m - (m >> 15)) | m);
}

}  // namespace

__global__ void __launch_bounds__(kBwdThreads)
k_cnn_bwd(const float *__restrict__ coef, const float *__restrict__ dcoef, CnnPlanes pl,
          CnnBwdBlocks bk, int H, int W, const uint16_t *__restrict__ W1k,
          const uint16_t *__restrict__ W2p, const uint16_t *__restrict__ W2tp,
          const uint16_t *__restrict__ W3p, const float *__restrict__ params,
          float *__restrict__ partial) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[kLdsBwd];
  const int lane = threadIdx.x & 63, n0 = lane & 15, g0 = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nb = wave & 1, strip = (wave >> 1) & 1, half = wave >> 2;
  const size_t HWn = (size_t)H * W;
  uint32_t *x0s = (uint32_t *)(smem + kOX0);
  // dz as pairs of bfloat16: element k holds dz[k] and dz[k + 1]
  uint32_t *dzs = (uint32_t *)(smem + kODZ);
  float *d3 = (float *)(smem + kODA);

  // this block's scale, its planes and tiles
  int j = 0;
  while (j + 1 < pl.J && (int)blockIdx.x >= bk.first[j + 1]) ++j;
  const int tiles_x = (W + BW - 1) / BW, per_plane = tiles_x * ((H + BH - 1) / BH);
  const int ntiles = (pl.start[j + 1] - pl.start[j]) * per_plane;
  const int step = bk.first[j + 1] - bk.first[j];
  const float *P = params + (size_t)j * kCnnParams;

  const int n = n0, g = g0;
  // ---- operands held for the whole kernel ----
  bf16x8 w1[2], w2[9], w2t[9], w3f, w3t[2];
  f32x4 bias1[2], bias2;
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    // layer 1, taps and channels on K: lane group g < 3 holds tap row g,
    // element 2 dx + c tap column dx of input channel c
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const bool used = g < 3 && e < 6;
      const uint16_t h = used ? packed_w1(W1k, j, 16 * b + n, e & 1, 3 * g + (e >> 1)) : (uint16_t)0;
      w1[b][e] = *(const __bf16 *)&h;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) bias1[b][e] = P[kOffB1 + 16 * b + 4 * g + e];
    // transposed layer 3, taps on K: channel 16 b + n; lane group g < 3 holds
    // the taps of row 2 - g, element e < 3 that of column 2 - e
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const bool used = g < 3 && e < 3;
      const uint16_t h = used ? *packed_w3(W3p, j, 16 * b + n, 8 - 3 * g - e) : (uint16_t)0;
      w3t[b][e] = *(const __bf16 *)&h;
    }
  }
#pragma unroll
  for (int t = 0; t < 9; ++t) {
    w2[t] = *(const bf16x8 *)(W2p + ((((size_t)j * 9 + t) * 2 + nb) * 64 + lane) * 8);
    w2t[t] = *(const bf16x8 *)(W2tp + ((((size_t)j * 9 + t) * 2 + nb) * 64 + lane) * 8);
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) bias2[e] = P[kOffB2 + 16 * nb + 4 * g + e];
  // layer 3 with the taps on M: row n = tap, k = channel
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const uint16_t h = n < 9 ? *packed_w3(W3p, j, 8 * g + e, n) : (uint16_t)0;
    w3f[e] = *(const __bf16 *)&h;
  }
  const float b3 = P[kOffB3];
  bf16x8 ones;
#pragma unroll
  for (int e = 0; e < 8; ++e) ones[e] = (__bf16)1.0f;

  // gradient accumulators: dW2 [tap] for channels (16 half + 4 g + e, 16 nb + n)
  // of this strip; dW1 [c] taps 4 g + e, channel 16 nb + n (row 9 of c = 1 sums
  // da1); dW3 channels 16 half + 4 g + e, tap n
  const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
  f32x4 g2[9], g1[2] = {zero4, zero4}, g3 = zero4, gb2 = zero4;
  float gb3 = 0.f;
#pragma unroll
  for (int t = 0; t < 9; ++t) g2[t] = zero4;

  struct Tile {
    int ty0, tx0, b, i;
  };
  auto tile_at = [&](int q) {
    Tile t;
    const int p = q / per_plane, r = q % per_plane;
    t.ty0 = (r / tiles_x) * BH;
    t.tx0 = (r % tiles_x) * BW;
    t.b = p / pl.nsub[j];
    t.i = pl.first[j] + p % pl.nsub[j];
    return t;
  };
  // coefficients of the x0 region and dL/dc' c of the dz region, in registers
  float xr[kXPer], pc[kZPer], pd[kZPer];
  auto fetch = [&](const Tile &t) {
    const size_t o = ((size_t)t.b * pl.R + t.i) * HWn;
    const float *cb = coef + o, *db = dcoef + o;
    const int tid = fresh(threadIdx.x);
#pragma unroll
    for (int u = 0; u < kXPer; ++u) {
      const int q = tid + u * kBwdThreads;
      const int r = (q * 1561) >> 16;                        // q / 42
      const int yy = t.ty0 - 5 + r, xx = t.tx0 - 5 + q - r * XW;
      const bool in = q < XH * XW && (unsigned)yy < (unsigned)H && (unsigned)xx < (unsigned)W;
      xr[u] = in ? cb[yy * W + xx] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < kZPer; ++u) {
      const int q = tid + u * kBwdThreads;
      const int r = (q * 1821) >> 16;                        // q / 36
      const int yy = t.ty0 - 2 + r, xx = t.tx0 - 2 + q - r * ZW;
      const bool in = q < ZH * ZW && (unsigned)yy < (unsigned)H && (unsigned)xx < (unsigned)W;
      pc[u] = in ? cb[yy * W + xx] : 0.f;
      pd[u] = in ? db[yy * W + xx] : 0.f;
    }
  };

  if (threadIdx.x < 4) *(uint32_t *)(smem + kOZero + 4 * threadIdx.x) = 0u;
  int q = (int)blockIdx.x - bk.first[j];
  Tile t = tile_at(q < ntiles ? q : 0);
  if (q < ntiles) fetch(t);
  for (; q < ntiles; q += step) {
    const int ty0 = t.ty0, tx0 = t.tx0;
    const bool interior = ty0 >= 5 && ty0 + BH + 5 <= H && tx0 >= 5 && tx0 + BW + 5 <= W;
    // ---- x0 of this tile ----
    float prod[kZPer];
    {
      const float sg = pl.sigma[t.b], den = sg * pl.l2[t.i];
      const uint32_t ch1 = (uint32_t)f2bf(sg * (255.0f / 50.0f)) << 16;
      const int tx = fresh(threadIdx.x);
#pragma unroll
      for (int u = 0; u < kXPer; ++u) {
        const int k = tx + u * kBwdThreads;
        if (k >= XH * XW) continue;
        const int r = (k * 1561) >> 16;                      // k / 42
        const int yy = ty0 - 5 + r, xx = tx0 - 5 + k - r * XW;
        const bool in = (unsigned)yy < (unsigned)H && (unsigned)xx < (unsigned)W;
        x0s[k] = in ? ((uint32_t)f2bf(fabsf(xr[u]) / den) | ch1) : 0u;
      }
#pragma unroll
      for (int u = 0; u < kZPer; ++u) prod[u] = pd[u] * pc[u];
    }
    __syncthreads();

    // ---- layer 1 on T+4: three rows of 40 pixels per wave ----
    {
      const int n = fresh(n0), g = fresh(g0);
      static_assert(AH == 3 * NWV && AW == 40, "rows per wave");
      // pixel q of the wave's 120 (the last 8 lanes of block 7 repeat the last
      // pixel); lane group 3, whose weights are zero, reads zeros
      auto l1 = [&](int k0, auto count) {
        constexpr int S = decltype(count)::value;
        bf16x8 xb[S];
        int o[S];
        uint32_t in[S];
#pragma unroll
        for (int s = 0; s < S; ++s) {
          const int q = min(16 * (k0 + s) + n, 3 * AW - 1);
          const int rl = (q >= AW) + (q >= 2 * AW), c = q - rl * AW;
          const uint32_t *xp = (const uint32_t *)(smem + (g < 3 ? kOX0 + ((3 * wave + g) * XW + q + 2 * rl) * 4 : kOZero));
          xb[s] = frag(make_uint2(xp[0], xp[1]), make_uint2(xp[2], 0u));
          o[s] = kOH1 + (3 * wave * AW + q) * kPix + (swz(c, g >> 1) | (g & 1) * 8);
          in[s] = 0xFFFFFFFFu;
          if (!interior) {
            const int yy = ty0 - 4 + 3 * wave + rl, xx = tx0 - 4 + c;
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
      l1(0, IntC<4>{});
      l1(4, IntC<4>{});
    }
    __syncthreads();

    // ---- layer 2 on T+3 (channels 16 nb ..): columns 0..31 in two strips of
    // two halves of 11 rows, streamed; the other 6 columns in blocks of 16 ----
    {
      constexpr int RH = EH / 2;
      static_assert(EH % 2 == 0 && EW - 32 == 6, "strip geometry");
      const int n = fresh(n0), g = fresh(g0);
      const int r0 = RH * half, c = 16 * strip + n;
      int ad[3];
#pragma unroll
      for (int dx = 0; dx < 3; ++dx)
        ad[dx] = kOH1 + (r0 * AW + c + dx) * kPix + swz(c + dx, g);
      const int st = kOH2 + (r0 * EW + c) * kPix + swz(c, 2 * nb + (g >> 1)) + (g & 1) * 8;
      const bool cin = (unsigned)(tx0 - 3 + c) < (unsigned)W;
      f32x4 acc[3];
      bf16x8 fr[2][3];
#pragma unroll
      for (int dx = 0; dx < 3; ++dx) fr[0][dx] = *(const bf16x8 *)(smem + ad[dx]);
#pragma unroll
      for (int y = 0; y < RH + 2; ++y) {
        if (y + 1 < RH + 2) {
#pragma unroll
          for (int dx = 0; dx < 3; ++dx)
            fr[(y + 1) & 1][dx] = *(const bf16x8 *)(smem + ad[dx] + (y + 1) * AW * kPix);
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
          const int yy = ty0 - 3 + r0 + y - 2;
          const uint32_t in = (cin && (unsigned)yy < (unsigned)H) ? 0xFFFFFFFFu : 0u;
          *(uint2 *)(smem + st + (y - 2) * EW * kPix) = relu_pack(acc[(y - 2) % 3], in);
        }
      }
      // (22 rows of 6 pixels: blocks wave / 2, + 4 and, for the first pair of
      // waves, + 8)
      constexpr int NL = EH * 6;
      static_assert((NL + 15) / 16 == 9, "blocks of the remaining columns");
      auto rest = [&](int b0, auto count) {
        constexpr int S = decltype(count)::value;
        f32x4 a[S];
        int o[S][3], so[S];
        uint32_t in[S];
#pragma unroll
        for (int s = 0; s < S; ++s) {
          // (lanes past the last pixel repeat it)
          const int l = min((b0 + 4 * s) * 16 + n, NL - 1);
          const int r = (l * 10923) >> 16, cl = 32 + l - 6 * r;   // l / 6
          in[s] = 0xFFFFFFFFu;
          if (!interior) {
            const int yy = ty0 - 3 + r, xx = tx0 - 3 + cl;
            in[s] = ((unsigned)yy < (unsigned)H && (unsigned)xx < (unsigned)W) ? 0xFFFFFFFFu : 0u;
          }
#pragma unroll
          for (int dx = 0; dx < 3; ++dx) o[s][dx] = kOH1 + (r * AW + cl + dx) * kPix + swz(cl + dx, g);
          so[s] = kOH2 + (r * EW + cl) * kPix + swz(cl, 2 * nb + (g >> 1)) + (g & 1) * 8;
          a[s] = bias2;
        }
#pragma unroll
        for (int k = 0; k < 9; ++k)
#pragma unroll
          for (int s = 0; s < S; ++s)
            a[s] = mma(w2[k], *(const bf16x8 *)(smem + o[s][k % 3] + (k / 3) * AW * kPix), a[s]);
#pragma unroll
        for (int s = 0; s < S; ++s) *(uint2 *)(smem + so[s]) = relu_pack(a[s], in[s]);
      };
      rest(wave >> 1, IntC<2>{});
      if (wave < 2) rest(8, IntC<1>{});
    }
    __syncthreads();

    // ---- layer 3: D[tap][p] = sum_ci W3[ci][tap] h2[p][ci] on T+3 ----
    // (rows wave, wave + 8, wave + 16 in blocks of 16, 16 and 6 pixels)
    {
      const int n = fresh(n0), g = fresh(g0);
      const int cl = min(32 + n, EW - 1);
      const int hc[3] = {n * kPix + swz(n, g), (16 + n) * kPix + swz(16 + n, g), cl * kPix + swz(cl, g)};
      const int dc[3] = {n, 16 + n, cl};
      f32x4 d[3][3];
#pragma unroll
      for (int rr = 0; rr < 3; ++rr) {
        const int r = min(wave + NWV * rr, EH - 1);
#pragma unroll
        for (int k = 0; k < 3; ++k)
          d[rr][k] = mma(w3f, *(const bf16x8 *)(smem + kOH2 + r * EW * kPix + hc[k]), zero4);
      }
      // lane group g holds taps 4 g ..: 4, 4 and 1 of them are used
      if (g < 3) {
#pragma unroll
        for (int rr = 0; rr < 3; ++rr)
#pragma unroll
          for (int k = 0; k < 3; ++k)
            d3[4 * g * NE + min(wave + NWV * rr, EH - 1) * EW + dc[k]] = d[rr][k][0];
      }
      if (g < 2) {
#pragma unroll
        for (int rr = 0; rr < 3; ++rr)
#pragma unroll
          for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int e = 1; e < 4; ++e)
              d3[(4 * g + e) * NE + min(wave + NWV * rr, EH - 1) * EW + dc[k]] = d[rr][k][e];
      }
    }
    __syncthreads();

    // ---- gain and dz = dL/dc' c g (1 - g) on T+2 ----
    {
      const int tid = fresh(threadIdx.x);
#pragma unroll
      for (int u = 0; u < kZPer; ++u) {
        const int k = tid + u * kBwdThreads;
        if (k < ZH * ZW) {
          const int r = (k * 1821) >> 16, c = k - r * ZW;   // k / 36
          float z = b3;
#pragma unroll
          for (int e = 0; e < 9; ++e) z += d3[k + 2 * r + e * NE + (e / 3) * EW + e % 3];
          const float gv = 1.0f / (1.0f + __expf(-z));
          const int yy = ty0 - 2 + r, xx = tx0 - 2 + c;
          const bool in = (unsigned)yy < (unsigned)H && (unsigned)xx < (unsigned)W;
          const uint16_t v = in ? f2bf(prod[u] * gv * (1.f - gv)) : (uint16_t)0;
          ((uint16_t *)dzs)[2 * k] = v;
          if (k > 0) ((uint16_t *)dzs)[2 * k - 1] = v;
          if (r >= 2 && r < 2 + BH && c >= 2 && c < 2 + BW) gb3 += bf2f(v);
        }
      }
    }
    __syncthreads();

    // ---- da2 = [h2 > 0] (W3 transposed) dz on T+1, taps on K ----
    // lane group g < 3 reads the three dz of row r + g of T+2 (columns c ..);
    // lanes past the last pixel repeat it
    {
      const int n = fresh(n0), g = fresh(g0);
      auto l3t = [&](int b0, auto count) {
        constexpr int S = decltype(count)::value;
        bf16x8 zb[S];
        uint2 h[S][2];
        int o[S];
#pragma unroll
        for (int s = 0; s < S; ++s) {
          const int p = min((b0 + NWV * s) * 16 + n, DH * DW - 1);
          const int r = (p * 1928) >> 16, c = p - DW * r;     // p / 34
          const uint32_t *zp = (const uint32_t *)(smem + (g < 3 ? kODZ + (p + 2 * r + g * ZW) * 4 : kOZero));
          zb[s] = frag(make_uint2(zp[0], zp[2] & 0xFFFFu), make_uint2(0u, 0u));
          const int ho = kOH2 + (p + 4 * r + 2 * EW + 2) * kPix + (swz(c + 2, g >> 1) | (g & 1) * 8);
          h[s][0] = *(const uint2 *)(smem + ho);
          h[s][1] = *(const uint2 *)(smem + (ho ^ 32));
          o[s] = kODA + p * kPix + (swz(c, g >> 1) | (g & 1) * 8);
        }
        f32x4 d[S][2];
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
          for (int b = 0; b < 2; ++b) d[s][b] = mma(w3t[b], zb[s], zero4);
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
          for (int b = 0; b < 2; ++b) {
            const uint2 w = pack4(d[s][b]);
            *(uint2 *)(smem + (b ? o[s] ^ 32 : o[s])) =
                make_uint2(keep_nonzero(w.x, h[s][b].x), keep_nonzero(w.y, h[s][b].y));
          }
      };
      static_assert((DH * DW + 15) / 16 <= 5 * NWV, "blocks of da2");
      l3t(wave, IntC<3>{});
      l3t(wave + 3 * NWV, IntC<2>{});
    }
    // the next tile's coefficients land during the gradient products below
    const Tile tn = tile_at(q + step < ntiles ? q + step : q);
    if (q + step < ntiles) fetch(tn);
    __syncthreads();

    // ---- da1 = [h1 > 0] (W2 transposed) da2 on T: rows 8 half .. of the
    // strip, the pixels on M, so that a lane holds 4 pixels of channel
    // 16 nb + n: two rows make the pixel operand of dW1 in registers ----
    {
      constexpr int RH = BH / 2;
      const int n = fresh(n0), g = fresh(g0);
      const int r0 = RH * half, c = 16 * strip + n;
      int ad[3];
#pragma unroll
      for (int dx = 0; dx < 3; ++dx)
        ad[dx] = kODA + (r0 * DW + c + dx) * kPix + swz(c + dx, g);
      const int xm = 16 * strip + 4 * g + 4;       // h1 column of pixel 4 g
      const int hm = kOH1 + ((r0 + 4) * AW + xm) * kPix + swz(xm, 2 * nb + (n >> 3)) + (n & 7) * 2;
      const int tap = n < 9 ? n : 8;
      const uint32_t *xp = x0s + (r0 + 4 + tap / 3) * XW + 16 * strip + 4 * g + 4 + tap % 3;
      f32x4 acc[3];
      bf16x8 fr[2][3];
      uint2 prev = make_uint2(0u, 0u);
#pragma unroll
      for (int dx = 0; dx < 3; ++dx) fr[0][dx] = *(const bf16x8 *)(smem + ad[dx]);
#pragma unroll
      for (int y = 0; y < RH + 2; ++y) {
        if (y + 1 < RH + 2) {
#pragma unroll
          for (int dx = 0; dx < 3; ++dx)
            fr[(y + 1) & 1][dx] = *(const bf16x8 *)(smem + ad[dx] + (y + 1) * DW * kPix);
        }
        if (y < RH) acc[y % 3] = zero4;
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int dx = 0; dx < 3; ++dx)
#pragma unroll
          for (int dy = 2; dy >= 0; --dy) {
            const int r = y - dy;
            if (r >= 0 && r < RH) acc[r % 3] = mma(fr[y & 1][dx], w2t[3 * dy + dx], acc[r % 3]);
          }
        __builtin_amdgcn_s_setprio(0);
        if (y >= 2) {
          const int r = y - 2;
          f32x4 o;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const uint16_t h = *(const uint16_t *)(smem + (e < 2 ? hm : hm ^ 16) + (r * AW + e) * kPix);
            o[e] = h != 0 ? acc[r % 3][e] : 0.f;
          }
          const uint2 cur = pack4(o);
          if (r & 1) {
            const bf16x8 db = frag(prev, cur);
            uint2 c0[2], c1[2];
#pragma unroll
            for (int k = 0; k < 2; ++k) {
              uint32_t x[4];
#pragma unroll
              for (int e = 0; e < 4; ++e) x[e] = xp[(r - 1 + k) * XW + e];
              c0[k] = make_uint2(__builtin_amdgcn_perm(x[1], x[0], 0x05040100u),
                                 __builtin_amdgcn_perm(x[3], x[2], 0x05040100u));
              c1[k] = make_uint2(__builtin_amdgcn_perm(x[1], x[0], 0x07060302u),
                                 __builtin_amdgcn_perm(x[3], x[2], 0x07060302u));
              if (n == 9) c1[k] = make_uint2(0x3F803F80u, 0x3F803F80u);   // sums da1
            }
            g1[0] = mma(frag(c0[0], c0[1]), db, g1[0]);
            g1[1] = mma(frag(c1[0], c1[1]), db, g1[1]);
          }
          prev = cur;
        }
      }
    }

    // ---- dW2 of channels (16 half .., 16 nb ..) over the strip; dW3 of
    // channels 16 half .. (waves with nb = 1) ----
    {
      const int n = fresh(n0), g = fresh(g0);
      // lane i of a 16-lane group reads pixel 4 g + i / 4, channels 4 (i % 4) ..
      const int px = 16 * strip + 4 * g + (n >> 2), ch = n & 3;
      int ah[3];
#pragma unroll
      for (int dx = 0; dx < 3; ++dx) {
        const int x = px + 3 + dx;
        ah[dx] = kOH1 + (3 * AW + x) * kPix + swz(x, 2 * half + (ch >> 1)) + (ch & 1) * 8;
      }
      const int ab = kODA + (DW + px + 1) * kPix + swz(px + 1, 2 * nb + (ch >> 1)) + (ch & 1) * 8;
      const int ae = kOH2 + (3 * EW + px + 3) * kPix + swz(px + 3, 2 * half + (ch >> 1)) + (ch & 1) * 8;
      const int tap = n < 9 ? n : 8;
      const uint32_t *zp = dzs + (3 - tap / 3) * ZW + 16 * strip + 4 * g + 3 - tap % 3;
      auto tr = [&](int off) -> uint2 {
        const s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(smem + off));
        return *(const uint2 *)&v;
      };
      uint2 hr[4][3];
#pragma unroll
      for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int dx = 0; dx < 3; ++dx) hr[k][dx] = tr(ah[dx] + k * AW * kPix);
#pragma unroll
      for (int r = 0; r < BH; r += 2) {
        // h1 rows r + 3 .. r + 6 in hr[(row - 3) % 4]
#pragma unroll
        for (int k = 2; k < 4; ++k)
#pragma unroll
          for (int dx = 0; dx < 3; ++dx) hr[(r + k) & 3][dx] = tr(ah[dx] + (r + k) * AW * kPix);
        const bf16x8 db = frag(tr(ab + r * DW * kPix), tr(ab + (r + 1) * DW * kPix));
#pragma unroll
        for (int dy = 0; dy < 3; ++dy)
#pragma unroll
          for (int dx = 0; dx < 3; ++dx)
            g2[3 * dy + dx] = mma(frag(hr[(r + dy) & 3][dx], hr[(r + dy + 1) & 3][dx]), db, g2[3 * dy + dx]);
        if (half == 0) gb2 = mma(ones, db, gb2);
        if (nb == 1) {
          uint2 z[2];
#pragma unroll
          for (int k = 0; k < 2; ++k) z[k] = make_uint2(zp[(r + k) * ZW], zp[(r + k) * ZW + 2]);
          g3 = mma(frag(tr(ae + r * EW * kPix), tr(ae + (r + 1) * EW * kPix)), frag(z[0], z[1]), g3);
        }
      }
    }
    t = tn;
    __syncthreads();
  }

  // ---- the block's gradients, summed over its waves in a fixed order in LDS,
  // in the order of the parameter blob ----
  float *gs = (float *)(smem + kOH1);
  float *gw = (float *)(smem + kODZ);
  __syncthreads();
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) gb3 += __shfl_xor(gb3, o, 64);
  if (lane == 0) gw[wave] = gb3;
  for (int round = 0; round < 4; ++round) {
    // (round 0 writes every entry that a later round adds to)
    auto put = [&](int k, float v) { gs[k] = round == 0 ? v : gs[k] + v; };
    if (strip == round) {
#pragma unroll
      for (int tp = 0; tp < 9; ++tp)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          put(kOffW2 + ((16 * nb + n) * CH + 16 * half + 4 * g + e) * 9 + tp, g2[tp][e]);
      if (half == 0 && g == 0) put(kOffB2 + 16 * nb + n, gb2[0]);
      if (nb == 1 && n < 9) {
#pragma unroll
        for (int e = 0; e < 4; ++e) put(kOffW3 + (16 * half + 4 * g + e) * 9 + n, g3[e]);
      }
    }
    if (2 * strip + half == round) {
      const int co = 16 * nb + n;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (4 * g + e < 9) {
          put(kOffW1 + co * 18 + 4 * g + e, g1[0][e]);
          put(kOffW1 + co * 18 + 9 + 4 * g + e, g1[1][e]);
        }
      }
      if (g == 2) put(kOffB1 + co, g1[1][1]);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    float s = 0.f;
    for (int w = 0; w < NWV; ++w) s += gw[w];
    gs[kOffB3] = s;
  }
  __syncthreads();
  float *dst = partial + (size_t)blockIdx.x * kCnnParams;
  for (int k = threadIdx.x; k < kCnnParams; k += kBwdThreads) dst[k] = gs[k];
}

// grads[j][k] = sum of the partial gradients of scale j's blocks, in order
__global__ void __launch_bounds__(256)
k_cnn_bwd_sum(const float *__restrict__ partial, CnnBwdBlocks bk, float *__restrict__ grads) {
  const int k = blockIdx.x * 256 + threadIdx.x, j = blockIdx.y;
  if (k >= kCnnParams) return;
  float s = 0.f;
#pragma unroll 8
  for (int b = bk.first[j]; b < bk.first[j + 1]; ++b) s += partial[(size_t)b * kCnnParams + k];
  grads[(size_t)j * kCnnParams + k] = s;
}

// Blocks of each scale: one block per compute unit shared out by the number
// of tiles, at least one per scale and at most one per tile.
int cnn_bwd_blocks(const CnnPlanes &pl, int H, int W, int num_cu, CnnBwdBlocks &bk) {
  const long per = (long)((W + BW - 1) / BW) * ((H + BH - 1) / BH);
  const long total = per * pl.start[pl.J];
  bk.first[0] = 0;
  for (int j = 0; j < pl.J; ++j) {
    const long nt = per * (pl.start[j + 1] - pl.start[j]);
    long nblk = total > 0 ? nt * num_cu / total : 1;
    nblk = std::max(1L, std::min(nblk, nt));
    bk.first[j + 1] = bk.first[j] + (int)nblk;
  }
  return bk.first[pl.J];
}

hipError_t cnn_bwd(const float *coef, const float *dcoef, const CnnPlanes &pl, int H, int W,
                   const uint16_t *W1k, const uint16_t *W2p, const uint16_t *W2tp,
                   const uint16_t *W3p, const float *params, int num_cu, float *partial,
                   float *grads, hipStream_t st) {
  CnnBwdBlocks bk{};
  const int nblk = cnn_bwd_blocks(pl, H, W, num_cu, bk);
  hipLaunchKernelGGL(k_cnn_bwd, dim3(nblk), dim3(kBwdThreads), 0, st, coef, dcoef, pl, bk, H, W,
                     W1k, W2p, W2tp, W3p, params, partial);
  hipLaunchKernelGGL(k_cnn_bwd_sum, dim3((kCnnParams + 255) / 256, pl.J), dim3(256), 0, st,
                     partial, bk, grads);
  return hipGetLastError();
}

}  // namespace sl
