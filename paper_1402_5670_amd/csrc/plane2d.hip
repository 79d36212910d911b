// Whole-plane passes for small images (Algorithms 1 and 2): planes of 32, 48 or
// 64 lines by 32, 48 or 64 samples are transformed by one block in LDS, so a
// call takes one or two launches and the pair planes never reach memory.
//
// The line passes take 4 to 5 launches per direction, 2 to 4 us each, which is
// all the time of a small image, and write and re-read every pair plane.  Here
//   forward   block (group of pairs, image): row and column DFT of the image,
//             kept in registers; per pair filter product, column IDFT, row
//             IDFT, coefficient store.  The image's DFT is repeated per group,
//             half of one pair's work each.
//   inverse   block (group, image): per pair coefficient load, threshold, row
//             and column DFT, filter product, sum in registers, inverse
//             DFT of the sum: x, or with several groups a share of it that
//             k_plane2_sum adds, the lowpass's last.
//   denoise   both around the threshold, without coefficients.
// Measured on MI355X against the line passes, forward + inverse: one 64 x 64
// image 38 -> 17 us, 64 of them (R = 33) 76 -> 41 us; denoise of 8 such images
// 31 -> 14 us.  The line ends at 64 x 64: a larger plane is a longer chain for its
// block than the launches saved, and with many images the line passes' exchange
// costs less than repeating the image's DFT (R = 17, denoised, line passes and
// whole planes, us: 96 x 64, 1, 32 and 300 images 21.3, 45.0, 147 and 32.2, 43.7,
// 204; 64 x 96 21.1, 42.2, 139 and 27.7, 39.4, 166; 96 x 96 24.6, 51.7, 217 and
// 44.1, 68.1, 412; 128 x 128, both directions, R = 49, 1 and 30 images 38, 142 and
// 103, 195).  Only batches of 16 to 32 of the first two would gain.
//
// Plans, line FFTs and products are those of the line passes, applied to the
// same values, so results agree to float32 rounding.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "dispatch.hpp"
#include "fresh.hpp"
#include "tiles.hpp"

namespace sl {

namespace {

// Threads of a plane block: the most up to 512 that give every column (row) of
// a pass its own NTC (NTR) threads with no remainder.  A thread keeps its
// share of the spectrum (and of the sum) in registers over all pairs of the
// block.
template <int H, int W>
struct Plane2 {
  using PC = Plan<H>;
  using PR = Plan<W>;
  static constexpr int RL = row_lds_len<W>();
  static constexpr int NTC = PC::NT, EC = PC::E, NTR = PR::NT, ER = PR::E;
  static constexpr bool fits(int th) {
    return th % NTC == 0 && th % NTR == 0 && W % (th / NTC) == 0 && H % (th / NTR) == 0;
  }
  static constexpr int pick() {
    for (int th = 512; th >= 64; th -= 64)
      if (fits(th)) return th;
    return 0;
  }
  static constexpr int THREADS = pick();
  static constexpr int MC = THREADS / NTC, MR = THREADS / NTR;
  static constexpr int NCI = W / MC, NRI = H / MR;      // column, row iterations
  static constexpr size_t LDS = (size_t)H * RL * sizeof(float2);
  static constexpr bool WAVE = wave_lines<NTR>();
  // blocks per compute unit the registers should allow (waves per SIMD)
  static constexpr int WPE = (LDS <= 72 * 1024 ? 2 : 1) * ((THREADS + 255) / 256);
  static_assert(THREADS > 0 && LDS <= 150 * 1024, "plane shape");
};

template <int H, int W>
__device__ __forceinline__ LdsLine p2_col(float2 *pl, int x) {
  return LdsLine{pl + x + (x >> 3), Plane2<H, W>::RL};
}
template <int H, int W>
__device__ __forceinline__ LdsLine p2_row(float2 *pl, int y) {
  return LdsLine{pl + y * Plane2<H, W>::RL, 0};
}

// A block's LDS: the plane and the twiddles of both lengths (read there, they
// are not hoisted into registers across the pair loop).
template <int H, int W>
struct Plane2Lds {
  float2 pl[H * Plane2<H, W>::RL];
  float2 th[H], tw[W];
  __device__ __forceinline__ void stage(const float2 *__restrict__ gh, const float2 *__restrict__ gw) {
    for (int i = threadIdx.x; i < H; i += Plane2<H, W>::THREADS) th[i] = gh[i];
    for (int i = threadIdx.x; i < W; i += Plane2<H, W>::THREADS) tw[i] = gw[i];
  }
};

template <int H, int W>
using ColVals = float2[Plane2<H, W>::NCI][Plane2<H, W>::EC];

template <int H, int W, bool INV>
__device__ __forceinline__ void row_dft(float2 (&v)[(Plane2<H, W>::ER)], int t, const LdsLine &row,
                                        const Plane2Lds<H, W> &s) {
  fft_line_p<typename Plane2<H, W>::PR, INV, Plane2<H, W>::WAVE>(v, t, row, TwLds{s.tw});
}

// Spectrum of image b (columns in registers): row DFT of the real rows
// (MIX 1, 2: the inpainting input, as k_rows_real_fft), column DFT.  amax
// returns the thread's largest |x|.
template <int H, int W, int MIX>
__device__ __forceinline__ void p2_spectrum(Plane2Lds<H, W> &s,
                                            const float *__restrict__ x, const MixArgs &mix, int b,
                                            ColVals<H, W> &f, float &amax) {
  float2 *pl = s.pl;
  using PT = Plane2<H, W>;
  const int t = threadIdx.x % PT::NTR, m = threadIdx.x / PT::NTR;
  const size_t img = (size_t)b * H * W;
  amax = 0.f;
#pragma unroll
  for (int ri = 0; ri < PT::NRI; ++ri) {
    const int y = ri * PT::MR + m;
    float2 v[PT::ER];
#pragma unroll
    for (int e = 0; e < PT::ER; ++e) {
      const size_t i = img + (size_t)y * W + t + e * PT::NTR;
      float a;
      if constexpr (MIX == 0) {
        a = x[i];
      } else {
        const unsigned char known = mix.mask[i];
        const float fm = mix.fm[i], fe = MIX == 2 ? mix.f[i] : 0.f;
        a = known ? fm : fe;
      }
      v[e] = make_float2(a, 0.f);
      amax = fmaxf(amax, fabsf(a));
    }
    const LdsLine row = p2_row<H, W>(s.pl, y);
    row_dft<H, W, false>(v, t, row, s);
    line_sync<PT::WAVE>();
#pragma unroll
    for (int e = 0; e < PT::ER; ++e) row[t + e * PT::NTR] = v[e];
  }
  __syncthreads();
  const int mc = threadIdx.x % PT::MC, tc = threadIdx.x / PT::MC;
#pragma unroll
  for (int ci = 0; ci < PT::NCI; ++ci) {
    const LdsLine col = p2_col<H, W>(pl, ci * PT::MC + mc);
#pragma unroll
    for (int e = 0; e < PT::EC; ++e) f[ci][e] = col[tc + e * PT::NTC];
    fft_line_p<typename PT::PC, false>(f[ci], tc, col, TwLds{s.th});
  }
}

// Filter values of pair p at the thread's samples of column iteration ci (0 for
// the missing partner of an odd number of subbands)
template <int H, int W>
__device__ __forceinline__ void p2_filters(const float *__restrict__ filt, int p, int R, int ci,
                                           int o, float (&fa)[Plane2<H, W>::EC],
                                           float (&fb)[Plane2<H, W>::EC]) {
  using PT = Plane2<H, W>;
  const int ia = 2 * p, ib = ia + 1;
  const float *pa = filt + (size_t)ia * H * W, *pb = filt + (size_t)(ib < R ? ib : ia) * H * W;
#pragma unroll
  for (int e = 0; e < PT::EC; ++e) {
    fa[e] = pa[o + e * PT::NTC * W + ci * PT::MC];
    fb[e] = pb[o + e * PT::NTC * W + ci * PT::MC];
  }
  if (ib >= R) {
#pragma unroll
    for (int e = 0; e < PT::EC; ++e) fb[e] = 0.f;
  }
}

// pair plane: (psi_a + i psi_b) F, column IDFT, left in LDS (rows ready); fa,
// fb hold the filters of column iteration 0
template <int H, int W>
__device__ __forceinline__ void p2_pair_cols(Plane2Lds<H, W> &s, const ColVals<H, W> &f,
                                             const Plane2Args &a, int p,
                                             float (&fa)[Plane2<H, W>::EC],
                                             float (&fb)[Plane2<H, W>::EC]) {
  using PT = Plane2<H, W>;
  const int tid = fresh(threadIdx.x), mc = tid % PT::MC, tc = tid / PT::MC;
#pragma unroll
  for (int ci = 0; ci < PT::NCI; ++ci) {
    float2 v[PT::EC];
#pragma unroll
    for (int e = 0; e < PT::EC; ++e)
      v[e] = make_float2(f[ci][e].x * fa[e] - f[ci][e].y * fb[e],
                         f[ci][e].y * fa[e] + f[ci][e].x * fb[e]);
    if (ci + 1 < PT::NCI) p2_filters<H, W>(a.filt, p, a.R, ci + 1, tc * W + mc, fa, fb);
    const LdsLine col = p2_col<H, W>(s.pl, ci * PT::MC + mc);
    fft_line_p<typename PT::PC, true>(v, tc, col, TwLds{s.th});   // (leads with a barrier)
    __syncthreads();
#pragma unroll
    for (int e = 0; e < PT::EC; ++e) col[tc + e * PT::NTC] = v[e];
  }
  __syncthreads();
}

// acc += (psi_a - i psi_b) column DFT of the plane in LDS
template <int H, int W>
__device__ __forceinline__ void p2_acc_cols(Plane2Lds<H, W> &s, ColVals<H, W> &acc,
                                            const Plane2Args &a, int p) {
  using PT = Plane2<H, W>;
  const int tid = fresh(threadIdx.x), mc = tid % PT::MC, tc = tid / PT::MC;
#pragma unroll
  for (int ci = 0; ci < PT::NCI; ++ci) {
    float fa[PT::EC], fb[PT::EC];
    p2_filters<H, W>(a.filt, p, a.R, ci, tc * W + mc, fa, fb);
    const LdsLine col = p2_col<H, W>(s.pl, ci * PT::MC + mc);
    float2 v[PT::EC];
#pragma unroll
    for (int e = 0; e < PT::EC; ++e) v[e] = col[tc + e * PT::NTC];
    fft_line_p<typename PT::PC, false>(v, tc, col, TwLds{s.th});
#pragma unroll
    for (int e = 0; e < PT::EC; ++e) {
      acc[ci][e].x += fa[e] * v[e].x + fb[e] * v[e].y;
      acc[ci][e].y += fa[e] * v[e].y - fb[e] * v[e].x;
    }
  }
}

// Re IDFT(acc / Psi_hat) of the block's column sums: x for the only group of an
// image, else its share of x, real plane (b, g) of part.
//
// The transform is linear, so a group may finish its own share.  Shares are half
// the bytes of partial spectra and are added by as many blocks as there are
// samples for; adding the spectra of an image in the one block that transforms
// them took 11.3 us for a 64 x 64 image with 17 groups, against 2.5 us here for
// the transform and 2.7 us for the sum.
template <int H, int W>
__device__ __forceinline__ void p2_result(Plane2Lds<H, W> &s, ColVals<H, W> &acc,
                                          const Plane2Args &a, int b) {
  using PT = Plane2<H, W>;
  float2 *pl = s.pl;
  const int mc = threadIdx.x % PT::MC, tc = threadIdx.x / PT::MC;
#pragma unroll
  for (int ci = 0; ci < PT::NCI; ++ci) {
#pragma unroll
    for (int e = 0; e < PT::EC; ++e) {
      const float d = a.psi[(tc + e * PT::NTC) * W + ci * PT::MC + mc];
      acc[ci][e] = make_float2(acc[ci][e].x / d, acc[ci][e].y / d);
    }
    const LdsLine col = p2_col<H, W>(pl, ci * PT::MC + mc);
    fft_line_p<typename PT::PC, true>(acc[ci], tc, col, TwLds{s.th});
    __syncthreads();
#pragma unroll
    for (int e = 0; e < PT::EC; ++e) col[tc + e * PT::NTC] = acc[ci][e];
  }
  __syncthreads();
  const int t = threadIdx.x % PT::NTR, m = threadIdx.x / PT::NTR;
  float *xo = gridDim.x == 1 ? a.out + (size_t)b * H * W
                             : a.part + ((size_t)b * gridDim.x + blockIdx.x) * H * W;
#pragma unroll
  for (int ri = 0; ri < PT::NRI; ++ri) {
    const int y = ri * PT::MR + m;
    const LdsLine row = p2_row<H, W>(pl, y);
    float2 v[PT::ER];
#pragma unroll
    for (int e = 0; e < PT::ER; ++e) v[e] = row[t + e * PT::NTR];
    row_dft<H, W, true>(v, t, row, s);
#pragma unroll
    for (int e = 0; e < PT::ER; ++e) xo[y * W + t + e * PT::NTR] = v[e].x * a.inv_hw;
  }
}

// hard thresholds of a pair (0 = keep everything)
__device__ __forceinline__ void p2_thresholds(const ThrArgs &thr, float sg, int ia, int R,
                                              float &da, float &db) {
  const int ja = thr.jof[ia], ib = ia + 1;
  da = ja >= 0 ? (thr.K[ja] * sg) * thr.l2[ia] : 0.f;
  db = 0.f;
  if (ib < R) {
    const int jb = thr.jof[ib];
    if (jb >= 0) db = (thr.K[jb] * sg) * thr.l2[ib];
  }
}

}  // namespace

// ---- forward ----------------------------------------------------------------
// grid (groups, B); block g of an image takes pairs g, g + groups, ...
template <int H, int W, int DT>
__global__ void __launch_bounds__((Plane2<H, W>::THREADS), (Plane2<H, W>::WPE))
k_plane2_fwd(Plane2Args a, const float *__restrict__ x, typename Store<DT>::T *__restrict__ coef,
             float *__restrict__ scales) {
  using PT = Plane2<H, W>;
  using Raw = typename Store<DT>::Raw;
  __shared__ Plane2Lds<H, W> s;
  s.stage(a.twH, a.twW);
  __shared__ float red[PT::THREADS / 64];
  const int b = blockIdx.y, P = (a.R + 1) / 2;
  ColVals<H, W> f;
  float amax;
  const int o0 = (threadIdx.x / PT::MC) * W + threadIdx.x % PT::MC;
  float fa[PT::EC], fb[PT::EC];
  p2_filters<H, W>(a.filt, blockIdx.x, a.R, 0, o0, fa, fb);
  __syncthreads();   // twiddles
  p2_spectrum<H, W, 0>(s, x, MixArgs{}, b, f, amax);
  if constexpr (DT != 0) {
    amax = wave_max(amax);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = amax;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < PT::THREADS / 64; ++w) amax = fmaxf(amax, red[w]);
  }
  if (a.dual) {
    const int mc = threadIdx.x % PT::MC, tc = threadIdx.x / PT::MC;
#pragma unroll
    for (int ci = 0; ci < PT::NCI; ++ci)
#pragma unroll
      for (int e = 0; e < PT::EC; ++e) {
        const float d = a.psi[(tc + e * PT::NTC) * W + ci * PT::MC + mc];
        f[ci][e] = make_float2(f[ci][e].x / d, f[ci][e].y / d);
      }
  }
  for (int p = blockIdx.x; p < P; p += gridDim.x) {
    const int ia = 2 * p, ib = ia + 1;
    p2_pair_cols<H, W>(s, f, a, p, fa, fb);
    const int tid = fresh(threadIdx.x), t = tid % PT::NTR, m = tid / PT::NTR;
    // (lands during the rows below)
    if (p + (int)gridDim.x < P)
      p2_filters<H, W>(a.filt, p + gridDim.x, a.R, 0, (tid / PT::MC) * W + tid % PT::MC, fa, fb);
    float sa = a.inv_hw, sb = a.inv_hw;
    if constexpr (DT != 0) {
      // the storage scales, as k_cols_fft
      const float ba = amax * a.l1[ia], bb = ib < a.R ? amax * a.l1[ib] : 0.f;
      const float ca = ba > 0.f ? exp2f(ceilf(log2f(ba)) - 15.f) : 1.f;
      const float cb = bb > 0.f ? exp2f(ceilf(log2f(bb)) - 15.f) : 1.f;
      if (threadIdx.x == 0) {
        scales[(size_t)b * a.R + ia] = ca;
        if (ib < a.R) scales[(size_t)b * a.R + ib] = cb;
      }
      sa = a.inv_hw / ca;
      sb = a.inv_hw / cb;
    }
    Raw *pa = (Raw *)(coef + ((size_t)b * a.R + ia) * H * W);
    Raw *pb = (Raw *)(coef + ((size_t)b * a.R + (ib < a.R ? ib : ia)) * H * W);
#pragma unroll
    for (int ri = 0; ri < PT::NRI; ++ri) {
      const int y = ri * PT::MR + m;
      const LdsLine row = p2_row<H, W>(s.pl, y);
      float2 v[PT::ER];
#pragma unroll
      for (int e = 0; e < PT::ER; ++e) v[e] = row[t + e * PT::NTR];
      row_dft<H, W, true>(v, t, row, s);
#pragma unroll
      for (int e = 0; e < PT::ER; ++e)
        coef_store(pa + y * W + t + e * PT::NTR, Store<DT>::enc_raw(v[e].x * sa));
      if (ib < a.R) {
#pragma unroll
        for (int e = 0; e < PT::ER; ++e)
          coef_store(pb + y * W + t + e * PT::NTR, Store<DT>::enc_raw(v[e].y * sb));
      }
    }
  }
}

// ---- inverse ----------------------------------------------------------------
template <int H, int W, int DT>
__global__ void __launch_bounds__((Plane2<H, W>::THREADS), (Plane2<H, W>::WPE))
k_plane2_inv(Plane2Args a, const typename Store<DT>::T *__restrict__ coef,
             const float *__restrict__ scales, ThrArgs thr) {
  using PT = Plane2<H, W>;
  using Raw = typename Store<DT>::Raw;
  __shared__ Plane2Lds<H, W> s;
  s.stage(a.twH, a.twW);
  const int b = blockIdx.y, P = (a.R + 1) / 2;
  ColVals<H, W> acc;
#pragma unroll
  for (int ci = 0; ci < PT::NCI; ++ci)
#pragma unroll
    for (int e = 0; e < PT::EC; ++e) acc[ci][e] = make_float2(0.f, 0.f);
  Raw ra[PT::NRI][PT::ER], rb[PT::NRI][PT::ER];
  auto fetch = [&](int p) {
    const int tid = fresh(threadIdx.x), t = tid % PT::NTR, m = tid / PT::NTR;
    const int ia = 2 * p, ib = ia + 1;
    const Raw *pa = (const Raw *)(coef + ((size_t)b * a.R + ia) * H * W);
    const Raw *pb = (const Raw *)(coef + ((size_t)b * a.R + (ib < a.R ? ib : ia)) * H * W);
#pragma unroll
    for (int ri = 0; ri < PT::NRI; ++ri)
#pragma unroll
      for (int e = 0; e < PT::ER; ++e) {
        const int o = (ri * PT::MR + m) * W + t + e * PT::NTR;
        ra[ri][e] = coef_load(pa + o);
        rb[ri][e] = coef_load(pb + o);   // a valid plane; ignored without a partner
      }
  };
  fetch(blockIdx.x);
  for (int p = blockIdx.x; p < P; p += gridDim.x) {
    const int ia = 2 * p, ib = ia + 1;
    const bool has_b = ib < a.R;
    float sa = 1.f, sb = 1.f, da = 0.f, db = 0.f;
    if constexpr (DT != 0) {
      sa = scales[(size_t)b * a.R + ia];
      if (has_b) sb = scales[(size_t)b * a.R + ib];
    }
    if (thr.sigma) p2_thresholds(thr, thr.sigma[b], ia, a.R, da, db);
    __syncthreads();   // the previous pair's column pass has left LDS
    const int tid = fresh(threadIdx.x), t = tid % PT::NTR, m = tid / PT::NTR;
#pragma unroll
    for (int ri = 0; ri < PT::NRI; ++ri) {
      float2 v[PT::ER];
#pragma unroll
      for (int e = 0; e < PT::ER; ++e) {
        float c = Store<DT>::dec_raw(ra[ri][e]) * sa;
        float d = has_b ? Store<DT>::dec_raw(rb[ri][e]) * sb : 0.f;
        if (!(fabsf(c) >= da)) c = 0.f;
        if (!(fabsf(d) >= db)) d = 0.f;
        v[e] = make_float2(c, d);
      }
      const LdsLine row = p2_row<H, W>(s.pl, ri * PT::MR + m);
      row_dft<H, W, false>(v, t, row, s);
      line_sync<PT::WAVE>();
#pragma unroll
      for (int e = 0; e < PT::ER; ++e) row[t + e * PT::NTR] = v[e];
    }
    if (p + (int)gridDim.x < P) fetch(p + gridDim.x);
    __syncthreads();
    p2_acc_cols<H, W>(s, acc, a, p);
  }
  p2_result<H, W>(s, acc, a, b);
}

// ---- fused denoise ------------------------------------------------------------
template <int H, int W, int MIX>
__global__ void __launch_bounds__((Plane2<H, W>::THREADS), (Plane2<H, W>::WPE))
k_plane2_thr(Plane2Args a, const float *__restrict__ x, ThrArgs thr, MixArgs mix) {
  using PT = Plane2<H, W>;
  __shared__ Plane2Lds<H, W> s;
  s.stage(a.twH, a.twW);
  const int b = blockIdx.y, P = (a.R + 1) / 2;
  const float sg = MIX ? mix.delta_init[b] * mix.fac : thr.sigma[b];
  ColVals<H, W> f, acc;
  float amax;
  __syncthreads();   // twiddles
  p2_spectrum<H, W, MIX>(s, x, mix, b, f, amax);
#pragma unroll
  for (int ci = 0; ci < PT::NCI; ++ci)
#pragma unroll
    for (int e = 0; e < PT::EC; ++e) acc[ci][e] = make_float2(0.f, 0.f);
  for (int p = blockIdx.x; p < P; p += gridDim.x) {
    const int ia = 2 * p;
    const int tid = fresh(threadIdx.x), t = tid % PT::NTR, m = tid / PT::NTR;
    float fa[PT::EC], fb[PT::EC], da, db;
    p2_filters<H, W>(a.filt, p, a.R, 0, (tid / PT::MC) * W + tid % PT::MC, fa, fb);
    p2_thresholds(thr, sg, ia, a.R, da, db);
    p2_pair_cols<H, W>(s, f, a, p, fa, fb);
#pragma unroll
    for (int ri = 0; ri < PT::NRI; ++ri) {
      const LdsLine row = p2_row<H, W>(s.pl, ri * PT::MR + m);
      float2 v[PT::ER];
#pragma unroll
      for (int e = 0; e < PT::ER; ++e) v[e] = row[t + e * PT::NTR];
      row_dft<H, W, true>(v, t, row, s);
#pragma unroll
      for (int e = 0; e < PT::ER; ++e) {
        float c = v[e].x * a.inv_hw, d = ia + 1 < a.R ? v[e].y * a.inv_hw : 0.f;
        if (!(fabsf(c) >= da)) c = 0.f;
        if (!(fabsf(d) >= db)) d = 0.f;
        v[e] = make_float2(c, d);
      }
      row_dft<H, W, false>(v, t, row, s);
      line_sync<PT::WAVE>();
#pragma unroll
      for (int e = 0; e < PT::ER; ++e) row[t + e * PT::NTR] = v[e];
    }
    __syncthreads();
    p2_acc_cols<H, W>(s, acc, a, p);
  }
  p2_result<H, W>(s, acc, a, b);
}

// x = the shares of G groups, the first one last; n samples per image (grid
// (blocks, B)).  Blocks of one wave, a sample per lane: an image has few, and x
// may be aligned to 4 bytes only.
//
// The first group's share, the lowpass's, is about x itself: added first, every
// further addition would round at the size of x.  Relative error against 64 bits
// of one 64 x 64 image, R = 33: 1.36e-7 with the lowpass share first, 0.97e-7 now
// (1.14e-7 when partial spectra were added before one transform).
__global__ void __launch_bounds__(64)
k_plane2_sum(const float *__restrict__ part, float *__restrict__ x, int G, int n) {
  const int i = blockIdx.x * 64 + threadIdx.x;
  if (i >= n) return;
  const float *src = part + (size_t)blockIdx.y * G * n + i;
  const float low = src[0];
  float v = 0.f;
#pragma unroll 8
  for (int g = 1; g < G; ++g) v += src[(size_t)g * n];
  x[(size_t)blockIdx.y * n + i] = v + low;
}

static hipError_t launch_plane2_sum(const Plane2Args &a, int n, int G, int B, hipStream_t st) {
  hipLaunchKernelGGL(k_plane2_sum, dim3((n + 63) / 64, B), dim3(64), 0, st, a.part, a.out, G, n);
  return hipGetLastError();
}

// ---- launchers ------------------------------------------------------------------
#define SL_FOR_EACH_PLANE2(X) \
  X(32, 32) X(32, 48) X(48, 32) X(48, 48) X(32, 64) X(64, 32) X(48, 64) X(64, 48) X(64, 64)

bool plane2_supported(int H, int W) {
#define X(h, w) \
  if (H == h && W == w) return true;
  SL_FOR_EACH_PLANE2(X)
#undef X
  return false;
}

// Pair groups per image: blocks to fill the compute units as often as they
// hold a plane (LDS), at most one per pair.
static int plane2_groups(const Sys2D &s, int B, size_t lds, int blocks) {
  const int P = (s.R + 1) / 2;
  const int per_cu = std::max(1, std::min((int)(160 * 1024 / lds), blocks));
  const long slots = (long)per_cu * s.num_cu;
  const long per = std::max(1L, ((long)P * B + slots - 1) / slots);
  return (int)((P + per - 1) / per);
}

int plane2_inv_groups(const Sys2D &s, int B, size_t part_planes) {
  int G = 1;
#define X(h, w) \
  if (s.H == h && s.W == w) G = plane2_groups(s, B, sizeof(Plane2Lds<h, w>), Plane2<h, w>::WPE * 256 / Plane2<h, w>::THREADS);
  SL_FOR_EACH_PLANE2(X)
#undef X
  // as many of them as the scratch holds shares for
  const size_t fit = 2 * part_planes / B;
  if (!s.split_pairs || fit < 2) return 1;
  const int P = (s.R + 1) / 2, g = (int)std::min<size_t>(G, fit), per = (P + g - 1) / g;
  return (P + per - 1) / per;
}

static Plane2Args plane2_args(const Sys2D &s) {
  Plane2Args a{};
  a.R = s.R;
  a.filt = s.filt;
  a.psi = s.psi;
  a.l1 = s.l1;
  a.twH = s.twH;
  a.twW = s.twW;
  a.inv_hw = 1.0f / ((float)s.H * (float)s.W);
  return a;
}

hipError_t launch_plane2_fwd(const Sys2D &s, const float *x, void *coef, float *scales, int B,
                             bool dual, hipStream_t st) {
  Plane2Args a = plane2_args(s);
  a.dual = dual;
#define X(h, w)                                                                                  \
  if (s.H == h && s.W == w) {                                                                    \
    const dim3 grid(plane2_groups(s, B, sizeof(Plane2Lds<h, w>), Plane2<h, w>::WPE * 256 / Plane2<h, w>::THREADS), B);           \
    const dim3 block(Plane2<h, w>::THREADS);                                                     \
    if (s.dtype == 1)                                                                            \
      hipLaunchKernelGGL((k_plane2_fwd<h, w, 1>), grid, block, 0, st, a, x, (__half *)coef,      \
                         scales);                                                                \
    else if (s.dtype == 2)                                                                       \
      hipLaunchKernelGGL((k_plane2_fwd<h, w, 2>), grid, block, 0, st, a, x,                      \
                         (__hip_bfloat16 *)coef, scales);                                        \
    else                                                                                         \
      hipLaunchKernelGGL((k_plane2_fwd<h, w, 0>), grid, block, 0, st, a, x, (float *)coef,       \
                         scales);                                                                \
    return hipGetLastError();                                                                    \
  }
  SL_FOR_EACH_PLANE2(X)
#undef X
  return hipErrorInvalidValue;
}

hipError_t launch_plane2_inv(const Sys2D &s, const void *coef, const float *scales,
                             const ThrArgs &thr, float *x, float *part, int G, int B,
                             hipStream_t st) {
  Plane2Args a = plane2_args(s);
  a.out = x;
  a.part = part;
#define X(h, w)                                                                                  \
  if (s.H == h && s.W == w) {                                                                    \
    const dim3 grid(G, B), block(Plane2<h, w>::THREADS);                                         \
    if (s.dtype == 1)                                                                            \
      hipLaunchKernelGGL((k_plane2_inv<h, w, 1>), grid, block, 0, st, a, (const __half *)coef,   \
                         scales, thr);                                                           \
    else if (s.dtype == 2)                                                                       \
      hipLaunchKernelGGL((k_plane2_inv<h, w, 2>), grid, block, 0, st, a,                         \
                         (const __hip_bfloat16 *)coef, scales, thr);                             \
    else                                                                                         \
      hipLaunchKernelGGL((k_plane2_inv<h, w, 0>), grid, block, 0, st, a, (const float *)coef,    \
                         scales, thr);                                                           \
    const hipError_t e = hipGetLastError();                                                      \
    return e != hipSuccess || G == 1 ? e : launch_plane2_sum(a, h * w, G, B, st);                \
  }
  SL_FOR_EACH_PLANE2(X)
#undef X
  return hipErrorInvalidValue;
}

hipError_t launch_plane2_thr(const Sys2D &s, const float *x, const MixArgs *mix,
                             const ThrArgs &thr, float *out, float *part, int G, int B,
                             hipStream_t st) {
  Plane2Args a = plane2_args(s);
  a.out = out;
  a.part = part;
#define X(h, w)                                                                                  \
  if (s.H == h && s.W == w) {                                                                    \
    const dim3 grid(G, B), block(Plane2<h, w>::THREADS);                                         \
    if (!mix)                                                                                    \
      hipLaunchKernelGGL((k_plane2_thr<h, w, 0>), grid, block, 0, st, a, x, thr, MixArgs{});     \
    else if (mix->first)                                                                         \
      hipLaunchKernelGGL((k_plane2_thr<h, w, 1>), grid, block, 0, st, a, x, thr, *mix);          \
    else                                                                                         \
      hipLaunchKernelGGL((k_plane2_thr<h, w, 2>), grid, block, 0, st, a, x, thr, *mix);          \
    const hipError_t e = hipGetLastError();                                                      \
    return e != hipSuccess || G == 1 ? e : launch_plane2_sum(a, h * w, G, B, st);                \
  }
  SL_FOR_EACH_PLANE2(X)
#undef X
  return hipErrorInvalidValue;
}

}  // namespace sl
