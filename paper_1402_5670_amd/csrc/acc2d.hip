// Inverse accumulation pass with streamed tiles, columns of 256, 512 or 1024
// points (Algorithm 2): ACC += sum over pairs of (psi_a - i psi_b)
// columnDFT(U), the last chunk divided by Psi_hat and inverse transformed.
//
// k_cols_fft_acc keeps a column per group of threads spread over the block's
// waves, so each of its FFT exchanges is a block barrier, and loads the pair
// planes into the registers that the FFT needs, so a block has nothing in
// flight while it transforms.  With many blocks per compute unit's turn that
// is hidden by the memory rate; with few it is not.  Here
//   - a tile of the pair plane (COLS columns) goes from memory straight to LDS
//     (global_load_lds, 16 bytes a lane) while the previous tile is transformed
//     in the other of two buffers;
//   - a column's lanes lie in one wave, so the FFT's exchanges stay inside the
//     wave; a tile takes two block barriers;
//   - the products with the filters run on the tile's rows, with coalesced
//     filter loads, after the transformed tile went through LDS.
// Row n of a tile keeps its 16-byte chunk k (two columns) at k ^ h(n), h(n) =
// n ^ n/8 ^ n/64, which spreads the rows that one instruction touches
// (consecutive ones, or every 8th) over the banks; h is linear over disjoint
// bits, so the rows of one thread differ by constants.  The plans, products and
// sums are those of k_cols_fft_acc, with which it agrees to float32 rounding.
// Measured sides of the choice: acc_stream (kernels2d.hip).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>

#include "dispatch.hpp"
#include "fft_core.hpp"
#include "fresh.hpp"

namespace sl {

namespace {

template <int N>
struct DTile {
  static constexpr int EM = N == 1024 ? 2 : 1;     // a column in one wave
  using PL = Plan<N, EM>;
  static constexpr int NT = PL::NT, E = PL::E;
  static constexpr int COLS = N == 1024 ? 8 : 16;
  static constexpr int C = COLS / 2;               // 16-byte chunks per row
  static constexpr int RB = COLS * 8;              // bytes per row
  static constexpr int THREADS = COLS * NT;
  static constexpr int TILE = N * RB;              // bytes of a tile
  static constexpr int UPT = N * C / THREADS;      // chunks per thread
  static constexpr int RPU = THREADS / C;          // rows per step of a thread's chunks
  static constexpr int WPE = (2 * 2 * TILE <= 160 * 1024 ? 2 : 1) * ((THREADS + 255) / 256);
  static_assert(THREADS % 64 == 0 && UPT * THREADS == N * C, "tile shape");
};

// 16-byte offset (bytes) of h(n) within a row
template <int N>
__device__ __forceinline__ constexpr int hx(int n) {
  return ((n ^ (n >> 3) ^ (n >> 6)) & (DTile<N>::C - 1)) << 4;
}

// address of chunk k of row n = n0 + d, with the bits of n0 and d disjoint:
// a0 = dt_addr(n0, k)
template <int N>
__device__ __forceinline__ int dt_addr(int n, int k) {
  return n * DTile<N>::RB + ((k << 4) ^ hx<N>(n));
}
template <int N>
__device__ __forceinline__ int dt_step(int a0, int d) {
  return (a0 ^ hx<N>(d)) + d * DTile<N>::RB;
}

// Radix stage S of a column (fft_core.hpp's stages; exchanges inside the wave).
template <int N, int S_, bool INV>
__device__ __forceinline__ void col_stage(float2 (&v)[DTile<N>::E], int t, unsigned char *buf, int k,
                                          const float2 *tw) {
  using PL = typename DTile<N>::PL;
  constexpr int E = PL::E, NT = PL::NT, r = PL::radix(S_), p = PL::pbefore(S_), NB = E / r;
  float2 x[NB][r];
  if constexpr (S_ == 0) {
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int q = 0; q < r; ++q) x[b][q] = v[b + q * NB];
  } else {
    line_sync<true>();
    const int a0 = dt_addr<N>(t, k);
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int q = 0; q < r; ++q)
        x[b][q] = *(const float2 *)(buf + dt_step<N>(a0, b * NT + q * (N / r)));
  }
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int i = t + b * NT;
    if constexpr (p > 1) {
      const int kk = i % p;
#pragma unroll
      for (int q = 1; q < r; ++q) {
        const float2 w = tw[q * kk * (N / (p * r))];
        x[b][q] = INV ? cmulconj(x[b][q], w) : cmul(x[b][q], w);
      }
    }
    dft_r<r, INV>(x[b]);
  }
  if constexpr (S_ == PL::S - 1) {
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int q = 0; q < r; ++q) v[b + q * NB] = x[b][q];
  } else {
    if constexpr (S_ > 0) line_sync<true>();
    // row (i - i % p) r + i % p + q p of i = t + b NT, NT a multiple of p: the
    // parts of t, b and q occupy disjoint bits
    static_assert(NT % p == 0, "line plan");
    const int kk = t % p, a0 = dt_addr<N>((t - kk) * r + kk, k);
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int q = 0; q < r; ++q)
        *(float2 *)(buf + dt_step<N>(a0, b * NT * r + q * p)) = x[b][q];
  }
}

template <int N, bool INV, int S_ = 0>
__device__ __forceinline__ void col_stages(float2 (&v)[DTile<N>::E], int t, unsigned char *buf,
                                           int k, const float2 *tw) {
  if constexpr (S_ < DTile<N>::PL::S) {
    col_stage<N, S_, INV>(v, t, buf, k, tw);
    col_stages<N, INV, S_ + 1>(v, t, buf, k, tw);
  }
}

// DFT of every column of the tile in buf, in place: the NT lanes of a column
// read its rows, transform and write them back.  The caller synchronises the
// block before and after.
template <int N, bool INV>
__device__ __forceinline__ void tile_dft(unsigned char *buf, const float2 *tw) {
  constexpr int E = DTile<N>::E, NT = DTile<N>::NT;
  const int tid = fresh(threadIdx.x), t = tid % NT, col = tid / NT, k = col >> 1;
  unsigned char *bc = buf + (col & 1) * 8;
  const int a0 = dt_addr<N>(t, k);
  float2 v[E];
#pragma unroll
  for (int e = 0; e < E; ++e) v[e] = *(const float2 *)(bc + dt_step<N>(a0, e * NT));
  line_sync<true>();
  col_stages<N, INV>(v, t, bc, k, tw);
  line_sync<true>();
#pragma unroll
  for (int e = 0; e < E; ++e) *(float2 *)(bc + dt_step<N>(a0, e * NT)) = v[e];
}

// Start moving a tile from memory to LDS: src is the tile's first row (wave
// uniform), W the row length in elements; the thread's chunk u is row
// tid / C + u RPU, LDS position tid % C, which holds source chunk
// (tid % C) ^ h(row).  No register receives data; the tile is complete after
// vmcnt(0) of every wave and a barrier.
template <int N>
__device__ __forceinline__ void tile_fetch(unsigned lds, const float2 *src, int W, unsigned v0) {
  using DT = DTile<N>;
  const unsigned wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
  for (int u = 0; u < DT::UPT; ++u) {
    const char *base = (const char *)src + (size_t)u * DT::RPU * W * 8;
    const unsigned v = (unsigned)fresh((int)v0) ^ (unsigned)hx<N>(u * DT::RPU);
    const unsigned m = lds + (unsigned)(u * DT::THREADS * 16) + wave * 1024u;
    asm volatile(
        "s_mov_b32 m0, %0\n\t"
        "s_nop 0\n\t"
        "global_load_lds_dwordx4 %1, %2 nt"
        :
        : "s"(m), "v"(v), "s"(base)
        : "memory", "m0");
  }
}
__device__ __forceinline__ void tile_wait() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

}  // namespace

// Grid (tiles x image groups, 1, pair groups), as acc_tile_group of the line
// pass flattens it: the blocks of one tile for every image group on one XCD.
template <int N, int BT>
__global__ void __launch_bounds__((DTile<N>::THREADS), (DTile<N>::WPE))
k_cols_acc_stream(const float2 *__restrict__ U, const float *__restrict__ filt,
               const float *__restrict__ psi, float2 *__restrict__ ACC, float2 *__restrict__ part,
               int Btot, int W, int R, int b0, int nb, int p0, int np, int first, int last,
               const float2 *__restrict__ tw) {
  using DT = DTile<N>;
  constexpr int UPT = DT::UPT, C = DT::C;
  __shared__ __attribute__((aligned(256))) unsigned char buf[2 * DT::TILE];
  // twiddles in LDS: a load from memory would wait for the tile under way
  __shared__ float2 twl[N];
  for (int i = threadIdx.x; i < N; i += DT::THREADS) twl[i] = tw[i];
  const int tiles = W / DT::COLS, groups = (int)gridDim.x / tiles;
  int tile, grp;
  if ((tiles & 7) == 0) {
    const int r = blockIdx.x & 7, u = blockIdx.x >> 3;
    grp = u % groups;
    tile = r * (tiles >> 3) + u / groups;
  } else {
    tile = blockIdx.x % tiles;
    grp = blockIdx.x / tiles;
  }
  const int col0 = tile * DT::COLS;
  const size_t plane = (size_t)N * W;
  // the thread's chunks: rows row0 + u RPU, columns col0 + 2 k, + 1
  const int row0 = threadIdx.x / C, k = threadIdx.x % C;
  const int a0 = dt_addr<N>(row0, k);
  const unsigned v0 = (unsigned)row0 * (unsigned)W * 8u + ((k << 4) ^ hx<N>(row0));
  const unsigned lo = ((unsigned)row0 * W + col0 + 2 * k) * 4u;   // bytes, float planes
  const size_t step4 = (size_t)DT::RPU * W * 4;
  const unsigned lds = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char *)buf;

  const int per = (np + (int)gridDim.z - 1) / (int)gridDim.z;
  const int q0 = (int)blockIdx.z * per, q1 = min(np, q0 + per);
  float2 *dst = blockIdx.z == 0 ? ACC : part + (size_t)(blockIdx.z - 1) * Btot * plane;
  float4 acc[BT][UPT];
#pragma unroll
  for (int bt = 0; bt < BT; ++bt) {
    const int bl = grp * BT + bt;
    const char *accp = (const char *)(dst + (size_t)(b0 + (bl < nb ? bl : 0)) * plane);
#pragma unroll
    for (int u = 0; u < UPT; ++u)
      acc[bt][u] = first ? make_float4(0.f, 0.f, 0.f, 0.f)
                         : *(const float4 *)(accp + 2 * (u * step4) + 2 * lo);
  }
  // tile (pair, image) in the order of the loop; the source of a missing last
  // image is the first one's plane (not stored)
  auto src = [&](int pp, int bt) {
    const int bl = grp * BT + bt;
    return U + ((size_t)(bl < nb ? bl : 0) * np + pp) * plane + col0;
  };
  int cur = 0;
  if (q0 < q1) tile_fetch<N>(lds, src(q0, 0), W, v0);
  for (int pp = q0; pp < q1; ++pp) {
    float2 fa[UPT], fb[UPT];
#pragma unroll
    for (int bt = 0; bt < BT; ++bt) {
      tile_wait();
      __syncthreads();      // the tile is complete; the other buffer is free
      if (bt == 0) {
        // the pair's filters, needed after the transform
        const int ia = 2 * (p0 + pp), ib = ia + 1;
        const char *pa = (const char *)(filt + (size_t)ia * plane);
        const char *pb = (const char *)(filt + (size_t)(ib < R ? ib : ia) * plane);
#pragma unroll
        for (int u = 0; u < UPT; ++u) {
          fa[u] = *(const float2 *)(pa + u * step4 + lo);
          fb[u] = *(const float2 *)(pb + u * step4 + lo);
        }
        if (ib >= R) {
#pragma unroll
          for (int u = 0; u < UPT; ++u) fb[u] = make_float2(0.f, 0.f);
        }
      }
      const int nbt = bt + 1 < BT ? bt + 1 : 0, npp = bt + 1 < BT ? pp : pp + 1;
      if (npp < q1) tile_fetch<N>(lds + (unsigned)((cur ^ 1) * DT::TILE), src(npp, nbt), W, v0);
      unsigned char *b = buf + cur * DT::TILE;
      tile_dft<N, false>(b, twl);
      __syncthreads();
      const int ar = fresh(a0);
#pragma unroll
      for (int u = 0; u < UPT; ++u) {
        const float4 v = *(const float4 *)(b + dt_step<N>(ar, u * DT::RPU));
        // (psi_a - i psi_b) * v
        acc[bt][u].x += fa[u].x * v.x + fb[u].x * v.y;
        acc[bt][u].y += fa[u].x * v.y - fb[u].x * v.x;
        acc[bt][u].z += fa[u].y * v.z + fb[u].y * v.w;
        acc[bt][u].w += fa[u].y * v.w - fb[u].y * v.z;
      }
      cur ^= 1;
    }
  }
#pragma unroll
  for (int bt = 0; bt < BT; ++bt) {
    const int bl = grp * BT + bt;
    if (last) {
      unsigned char *b = buf;
      __syncthreads();
#pragma unroll
      for (int u = 0; u < UPT; ++u) {
        const float2 d = *(const float2 *)((const char *)psi + u * step4 + lo);
        *(float4 *)(b + dt_step<N>(a0, u * DT::RPU)) =
            make_float4(acc[bt][u].x / d.x, acc[bt][u].y / d.x, acc[bt][u].z / d.y, acc[bt][u].w / d.y);
      }
      __syncthreads();
      tile_dft<N, true>(b, twl);
      __syncthreads();
#pragma unroll
      for (int u = 0; u < UPT; ++u) acc[bt][u] = *(const float4 *)(b + dt_step<N>(a0, u * DT::RPU));
    }
    if (bl < nb) {
      char *accp = (char *)(dst + (size_t)(b0 + bl) * plane);
#pragma unroll
      for (int u = 0; u < UPT; ++u) *(float4 *)(accp + 2 * (u * step4) + 2 * lo) = acc[bt][u];
    }
  }
}

#define SL_FOR_EACH_STREAM(X) X(256) X(512) X(1024)

int cols_acc_stream_cols(int H) {
#define X(N) \
  if (H == N) return DTile<N>::COLS;
  SL_FOR_EACH_STREAM(X)
#undef X
  return 0;
}

hipError_t launch_cols_acc_stream(const Sys2D &s, const float2 *U, float2 *ACC, float2 *part, int G,
                               int Btot, Chunk c, int bt, bool first, bool last, hipStream_t st) {
#define X(N)                                                                                     \
  if (s.H == N) {                                                                                \
    const dim3 grid(s.W / DTile<N>::COLS * ((c.nb + bt - 1) / bt), 1, G), block(DTile<N>::THREADS); \
    if (bt == 2)                                                                                 \
      hipLaunchKernelGGL((k_cols_acc_stream<N, 2>), grid, block, 0, st, U, s.filt, s.psi, ACC, part, \
                         Btot, s.W, s.R, c.b0, c.nb, c.p0, c.np, (int)first, (int)last, \
                         s.twH);                                                                 \
    else                                                                                         \
      hipLaunchKernelGGL((k_cols_acc_stream<N, 1>), grid, block, 0, st, U, s.filt, s.psi, ACC, part, \
                         Btot, s.W, s.R, c.b0, c.nb, c.p0, c.np, (int)first, (int)last, \
                         s.twH);                                                                 \
    return hipGetLastError();                                                                    \
  }
  SL_FOR_EACH_STREAM(X)
#undef X
  return hipErrorInvalidValue;
}

}  // namespace sl
