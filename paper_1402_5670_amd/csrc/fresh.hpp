// A value that the compiler does not keep addresses of (internal).
#pragma once

#include <hip/hip_runtime.h>

namespace sl {

// The value of x, computed anew: addresses derived from it stay inside their
// phase of a loop instead of being kept in registers across it, where operands
// and accumulators that live through the loop leave no room (in the shrinkage
// network's backward kernel hoisted addresses spilled 79 registers, 12.0 against
// 8.1 ms per 4 x 512^2 training step).
__device__ __forceinline__ int fresh(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

}  // namespace sl
