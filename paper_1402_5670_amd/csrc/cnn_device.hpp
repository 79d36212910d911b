// Device helpers shared by the shrinkage network's kernels (internal).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "fresh.hpp"

namespace sl {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef short s16x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));

constexpr int CH = 32;                         // hidden channels

__device__ __forceinline__ uint16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);             // round to nearest even
  return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// Activations in LDS: 32 channels of a pixel in 64 bytes, 16-byte chunk c of
// the pixel in column x at chunk c ^ ((x / 2) % 4).  By the bank-conflict
// counter, 16-byte reads of 16 consecutive pixels and the transposing reads of
// 8-byte pieces are then free of conflicts (without the permutation, or with
// (x / 4) % 4, the former take twice the cycles).
constexpr int kPix = 64;
// byte offset of 16-byte chunk c of column x within its pixel
__device__ __forceinline__ int swz(int x, int c) { return (c << 4) ^ ((x << 3) & 48); }

// 4 values rounded to bfloat16 (round to nearest even)
__device__ __forceinline__ uint2 pack4(f32x4 d) {
  const bf16x2 a = __builtin_convertvector((f32x2){d[0], d[1]}, bf16x2);
  const bf16x2 b = __builtin_convertvector((f32x2){d[2], d[3]}, bf16x2);
  return make_uint2(*(const uint32_t *)&a, *(const uint32_t *)&b);
}

// relu of 4 values, rounded to bfloat16, ANDed with the in-image mask (a
// maximum with 0 of the 16-bit patterns as signed integers: negative values
// have the sign bit set)
__device__ __forceinline__ uint2 relu_pack(f32x4 d, uint32_t in) {
  uint2 u = pack4(d);
  const s16x2 z = {0, 0};
  const s16x2 a = __builtin_elementwise_max(*(const s16x2 *)&u.x, z);
  const s16x2 b = __builtin_elementwise_max(*(const s16x2 *)&u.y, z);
  return make_uint2(*(const uint32_t *)&a & in, *(const uint32_t *)&b & in);
}

__device__ __forceinline__ bf16x8 frag(uint2 a, uint2 b) {
  const uint4 u = make_uint4(a.x, a.y, b.x, b.y);
  return *(const bf16x8 *)&u;
}

__device__ __forceinline__ f32x4 mma(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

template <int V>
struct IntC {
  static constexpr int value = V;
};

}  // namespace sl
