// Rules by which a kernel, or a path within one, is chosen: plain arithmetic, also for a host compiler.
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

// Pieces of one pair that the streaming pass is cut into where a batch is small: as few as have at most 2^shift tiles, all alike to a tile.
// (Pieces of 2^shift tiles and a rest were long and short in turn where the contexts are alike, and with two per pair the long ones went to
// every other workgroup, that is to half the XCDs: 32 requests of 575-600 tokens, 8 heads, 34.6 us where equal ranges take 31.4 and
// these 31.4, of 730-760 36.7 / 38.4 / 34.7, of 1500-1560 58.1 / 60.4 / 55.9; fp8 with 40 rows 36.7 / 33.6 / 34.0.)
__host__ __device__ inline int pieces_of(int tiles, int shift) { return (tiles + (1 << shift) - 1) >> shift; }
// first tile of piece i; least = tiles / pieces (the first ones have a tile more)
__host__ __device__ inline int piece_begin(int tiles, int pieces, int least, int i) {
  const int longer = tiles - least * pieces;
  return i * least + (i < longer ? i : longer);
}
// Partial slots: piece i of the pair that begins at unit u0 has pair + first_slot + i.  Distinct: a pair has at most (tiles >> shift) + 1 pieces,
// and the next one, tiles units on, begins at least (tiles >> shift) + 1 slots later.
__host__ __device__ inline int first_slot(int u0, int shift) { return u0 >> shift; }

// Whether the rows of a draft step bypass the Infinity Cache (non-temporal loads).  Rows that are there no more when they are next
// needed are read 7 to 14 % faster that way: 128 requests with lists of 256 31.3 / 27.1 us, 32 12.1 / 11.0, 16 of 1024 rows 21.3 / 19.4, fp8
// 64 of 512 22.2 / 20.7, each over so many pools that nothing stays cached; and the unified batch of 128 of 1-8 K tokens takes 154 / 144.
// But a layer that is verified or drafted from again before 256 MB have been read loses what is still there: one draft step and
// one verification of 32 requests of 4096 tokens in turn (34 MB of rows) 131 / 135.5, fp8 lists of 512 over three pools (67 MB each) 20.1 /
// 20.9.  So the line lies where two calls' rows no longer fit beside what the pass leaves: 96 MB.  (Above it, too, a single layer stepped
// over and over on the same pools reads less from memory without: 128 requests of 1-8 K tokens, verification and draft 586.5 / 593.5,
// unified batch 151 / 161.  A model has many layers between two steps of one.)
// list_rows: the host knows only what the index buffers have room for; where that is beyond the line, each workgroup asks again as if all lists
// were as long as its own.  (With lists of 256 and room for 2048, one draft step and one verification of 32 requests of 4096 tokens took
// 145 us when the room decided, 142 so, 140 without bypass.  All counts added up by every workgroup: 128 requests 30.6 us instead of 28.0,
// 300 with lists of 64 27 instead of 22.)
__host__ __device__ inline bool draft_bypasses(int64_t list_rows, bool fp8) { return list_rows * (fp8 ? 256 : 512) > (int64_t{96} << 20); }

}  // namespace pillar
