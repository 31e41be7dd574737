// Rules by which a launch is chosen, as plain arithmetic, also for a host compiler.
#pragma once

#include <algorithm>
#include <cstdint>

namespace pillar {

// Workgroups of the finish kernel that put O of one pair together and do nothing else: where half the chip would idle, as many as it holds
// beside the others (one per pair and 8192 tokens) in two rounds.  The rule must not ask for the statistic: with and without it, O has
// the same bits.  Without / with them, whole call: one request of 2100 tokens 26.4 / 23.5 us, 24 of 5-3000 24.1 / 20.4, 16 of 2-4 K with 8
// heads 60.7 / 57.0, 24 of 10-3000 with 64 rows 35.0 / 27.0, one of 32 K 64.4 / 56.0, one of 8 K without the statistic 41.1 / 30.3.
// With every compute unit taken by the statistic they only get in its way: 16 requests of 24-32 K tokens 494 / 496; and so they do where
// they take more than two turns of 1024 threads.  8 heads, 480-720 tokens: 64 rows, 80 pairs (two turns) 30.2 / 29.9, 88 30.9 / 34.0, 96
// 35.8 / 39.1; 1200-1800 tokens 46.0 / 42.7, 49.0 / 50.0, 49.9 / 51.7; 128 pairs of 768 with 36 rows 36.4 / 38.7 (with 20, 64 to 2048
// tokens 23.5 / 21.9).  Two turns may still lose a little: 48 rows, 96 pairs 33.4 / 34.5, 46.0 / 45.9.
// (max_seq_len is a bound: a caller whose contexts are shorter has fewer mergers than would pay, never more.)
inline int merger_groups(int64_t pairs, int max_seq_len, int rows, int threads, int num_cus) {
  const int64_t others = pairs * ((max_seq_len + int64_t{8191}) / 8192);
  if (2 * others > num_cus) return 0;
  const int at_once = 4 * (threads / 512);                               // rows of a turn
  const int room = static_cast<int>(2 * (num_cus - others) / pairs);
  if (rows > 16 * room) return 0;
  return std::min(room, (rows + at_once - 1) / at_once);
}

}  // namespace pillar
