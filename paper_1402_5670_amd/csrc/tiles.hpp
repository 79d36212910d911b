// Column tiles, coefficient storage types and in-LDS plane tiles shared by the
// 2D kernels (internal).
#pragma once

#include <hip/hip_bf16.h>
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include "fft_core.hpp"

namespace sl {

// Column tiles: M adjacent columns per block; with SL_COL_EMUL > 1 each thread
// of a column pass owns SL_COL_EMUL times more values, halving the threads per
// column and doubling the columns per block (wider coalesced segments) for
// lengths 256..512.
#ifndef SL_COL_EMUL
#define SL_COL_EMUL 1
#endif
template <int N>
struct CTile {
  static constexpr int EM = (N >= 256 && N <= 512) ? SL_COL_EMUL : 1;
  using PL = Plan<N, EM>;
  static constexpr int NT = PL::NT;
  static constexpr int E = PL::E;
  static constexpr int M = (NT * 16 <= 1024 ? 16 : 8) * (EM > 1 ? 2 : 1);
  static constexpr int THREADS = M * NT;
};

// ---------------------------------------------------------------------------
// storage encode / decode
// ---------------------------------------------------------------------------
template <int DT>
struct Store;
// T is the element type of the coefficient tensor; Raw its bit pattern as a
// plain scalar (kernels load and store Raw values, so that all loads of a row
// can be issued before the first conversion).
template <>
struct Store<0> {
  using T = float;
  using Raw = float;
  __device__ static T enc(float v) { return v; }
  __device__ static float dec(T v) { return v; }
  __device__ static Raw enc_raw(float v) { return v; }
  __device__ static float dec_raw(Raw v) { return v; }
};
template <>
struct Store<1> {
  using T = __half;
  using Raw = unsigned short;
  __device__ static T enc(float v) { return __float2half_rn(v); }
  __device__ static float dec(T v) { return __half2float(v); }
  __device__ static Raw enc_raw(float v) { return __half_as_ushort(__float2half_rn(v)); }
  __device__ static float dec_raw(Raw v) { return __half2float(__ushort_as_half(v)); }
};
template <>
struct Store<2> {
  using T = __hip_bfloat16;
  using Raw = unsigned short;
  __device__ static T enc(float v) { return __float2bfloat16(v); }
  __device__ static float dec(T v) { return __bfloat162float(v); }
  __device__ static Raw enc_raw(float v) { return __bfloat16_as_ushort(__float2bfloat16(v)); }
  __device__ static float dec_raw(Raw v) { return __uint_as_float((unsigned)v << 16); }
};

// Coefficient planes are streamed once per call; with SL_NT_COEF the float32
// coefficient stores and loads carry the non-temporal hint so that they do
// not displace the pass intermediates from the caches.
#ifndef SL_NT_COEF
#define SL_NT_COEF 0
#endif
template <class T>
__device__ __forceinline__ void coef_store(T *p, T v) {
  if constexpr (SL_NT_COEF && sizeof(T) == 4) __builtin_nontemporal_store(v, p);
  else *p = v;
}
template <class T>
__device__ __forceinline__ T coef_load(const T *p) {
  if constexpr (SL_NT_COEF && sizeof(T) == 4) return __builtin_nontemporal_load(p);
  else return *p;
}

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}

// Maximum over a block of THREADS threads, through lds (a wave's value each,
// or a thread's where the last wave is partial), which must not be in use and
// is free again only after the caller's next barrier.
template <int THREADS>
__device__ __forceinline__ float block_max(float v, float *lds) {
  constexpr bool FULL = THREADS % 64 == 0;
  constexpr int n = FULL ? THREADS / 64 : THREADS;
  if constexpr (FULL) v = wave_max(v);
  if (!FULL || (threadIdx.x & 63) == 0) lds[FULL ? threadIdx.x >> 6 : threadIdx.x] = v;
  __syncthreads();
  float mm = lds[0];
  for (int i = 1; i < n; ++i) mm = fmaxf(mm, lds[i]);
  return mm;
}

}  // namespace sl
