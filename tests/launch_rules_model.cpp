// Prints the launch rules of the 2D passes (csrc/launch_rules.hpp) for
// test_launch_rules.py.
#include <cstdio>

#include <hip/hip_runtime.h>

// An occupancy query that fails and leaves its error, as the runtime's does.
static hipError_t pending = hipSuccess;
template <class K>
static hipError_t failing_query(int *, K, int, size_t) {
  return pending = hipErrorInvalidValue;
}
static hipError_t take_error() {
  const hipError_t e = pending;
  pending = hipSuccess;
  return e;
}
#define hipOccupancyMaxActiveBlocksPerMultiprocessor failing_query
#define hipGetLastError take_error

#include "launch_rules.hpp"

template <int N>
static void rows() {
  std::printf("rows %d %d %d\n", N, sl::Tile<N>::M, sl::few_rows<N>());
}

__global__ void k_nothing() {}

int main() {
  rows<8>(), rows<12>(), rows<16>(), rows<24>(), rows<32>(), rows<48>(), rows<64>(), rows<96>();
  rows<128>(), rows<192>(), rows<256>(), rows<384>(), rows<512>(), rows<768>(), rows<1024>();
  const long blocks = sl::resident_blocks<k_nothing>(64, 256);
  std::printf("resident %ld %d\n", blocks, (int)hipGetLastError());
  for (long blocks : {256, 384, 512, 1024, 1030})
    std::printf("forward %ld %d\n", blocks, sl::forward_split(blocks, 1024, 256, 9));
  return 0;
}
