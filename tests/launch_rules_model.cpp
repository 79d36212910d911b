// Prints the launch rules of the 2D passes (csrc/launch_rules.hpp) for
// test_launch_rules.py.
#include <cstdio>

#include "launch_rules.hpp"

template <int N>
static void rows() {
  std::printf("rows %d %d %d\n", N, sl::Tile<N>::M, sl::few_rows<N>());
}

int main() {
  rows<8>(), rows<12>(), rows<16>(), rows<24>(), rows<32>(), rows<48>(), rows<64>(), rows<96>();
  rows<128>(), rows<192>(), rows<256>(), rows<384>(), rows<512>(), rows<768>(), rows<1024>();
  return 0;
}
