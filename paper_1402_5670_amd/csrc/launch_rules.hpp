// Block shapes and grid splits of the 2D passes (internal, host side).
#pragma once

#include <hip/hip_runtime.h>

#include <atomic>

#include "fft_core.hpp"

namespace sl {

// Row tiles: M rows per block.
// EM (line plan): each thread holds EM times the plan's values, so a line
// takes EM times fewer threads (EM = 2 makes a 1024-point row one wavefront,
// whose radix exchanges need no block barrier); the coefficient row passes
// take it per system (sl_system_set_line_plan, autotuned for uneven
// batches), and so does the inverse accumulation of 1024-point columns
// (launch_cols_fft_acc); the other column passes keep EM = 1.
template <int N, int EM = 1>
struct Tile {
  using PL = Plan<N, EM>;
  static constexpr int NT = PL::NT;
  static constexpr int E = PL::E;
  static constexpr int M = NT >= 128 ? 8 : 16;     // lines per block
  static constexpr int THREADS = M * NT;
};

// Lines per block of the rows of single planes (k_rows_real_fft,
// k_rows_real_ifft) where tiles of Tile<N>::M lines are few: blocks of two
// waves, a quarter of the lines for rows of 256 to 384 samples, an eighth from
// 512 on, half for 128 and 192.  Shorter rows keep their tile, which is two waves
// or less.  With narrower column tiles as well (cols_fft): row and column pass of
// a 512^2 image 6.1 + 6.5 -> 4.7 + 4.8 us, 3 x 96 x 384 in fp16, both
// directions, 56.1 -> 54.4 us, 2 x 192 x 768 97.6 -> 92.9.  (Rows of up to 48
// samples in blocks of two waves, which take two to eight times the lines, for
// the inverse, R = 17: 96 x 16 11.5 us against 10.8, 512 x 48 20.5 against
// 19.6, 384 x 32 15.3 against 14.7.)  The forward passes take them below a quarter of
// a block per compute unit: between that and one block there is little to gain
// alone (3 x 96 x 384 54.3 against 54.7), and four classes in one captured graph,
// whose branches share the device, lose 0.7% (1936 against 1922 us).
template <int N>
constexpr int few_rows() {
  constexpr int two_waves = Tile<N>::NT >= 128 ? 1 : 128 / Tile<N>::NT;
  return two_waves < Tile<N>::M ? two_waves : Tile<N>::M;
}

// Blocks of a kernel resident on the device at once; the occupancy of a kernel
// instance is queried once (one block per compute unit if that fails).
template <auto K>
long resident_blocks(int threads, int num_cu) {
  static std::atomic<int> slot{-1};
  int per = slot.load(std::memory_order_relaxed);
  if (per < 0) {
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, K, threads, 0) != hipSuccess) {
      (void)hipGetLastError();   // or the next launch's check would report it
      n = 0;
    }
    n = n < 1 ? 1 : n;
    per = n;
    slot.store(per, std::memory_order_relaxed);
  }
  return (long)per * num_cu;
}

// Parts to split the loop of a grid over np pairs into: blocks run their whole
// loop in one round, so a grid that is not a multiple of the resident blocks
// leaves a partly idle last round (6 x 1024^2: 384 blocks on 256, two rounds for
// one and a half).  The split with the fewest rounds per unit of work wins, each
// part costing `extra` pairs on top of its own; a further part has to save 5%,
// since each re-reads or writes a tile.
inline int round_split(long blocks, long resident, int np, int extra, int cap) {
  int best = 1;
  double best_cost = 1e30;
  for (int sp = 1; sp <= cap && sp <= np; ++sp) {
    const long per = (np + sp - 1) / sp;
    if ((np + per - 1) / per != sp) continue;              // no empty part
    const double cost = (double)((blocks * sp + resident - 1) / resident) * (double)(per + extra);
    if (cost < 0.95 * best_cost) {
      best_cost = cost;
      best = sp;
    }
  }
  return best;
}

// Parts of the forward column pass's pair loop for a grid of at least a block per
// compute unit.  One that is resident at once with two blocks or more per
// compute unit keeps its memory busy, and a split only has its tiles of the
// spectrum read again and its planes written further apart: 16 x 96 x 1024
// denoised (R = 17) 173.6 us in two parts, 167.5 whole, 64 x 128^2 95.9 and 93.0,
// 32 x 128 x 256 100.5 and 97.2 (the forward alone 104.1 and 101.9, 57.0 and
// 57.5, 58.6 and 58.4; 24 x 192 x 384 loses, 100.7 and 103.4).
inline int forward_split(long blocks, long resident, int num_cu, int np) {
  if (blocks >= 2L * num_cu && blocks <= resident) return 1;
  return round_split(blocks, resident, np, 0, 8);
}

}  // namespace sl
