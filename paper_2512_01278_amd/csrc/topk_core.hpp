// Exact selection of the K largest keys held in registers by one workgroup (paper Section 4.1: Top-K on
// the averaged scores).  Shared by the stand-alone Top-K kernel and by the verification finish kernel,
// which selects straight from on-chip scores.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "common.hpp"

namespace pillar {
namespace {

// float -> unsigned key whose integer order is the float order
__device__ __forceinline__ uint32_t order_key(float f) {
  const uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Inclusive prefix sum over the 64 lanes of a wavefront on the vector ALU: shifts by 1, 2, 4, 8
// inside each row of 16 lanes, then the last lane of row 0/2 is broadcast into row 1/3 and the last
// lane of the lower half into the upper half (lanes shifted in from outside read 0).
__device__ __forceinline__ uint32_t wave_inclusive_sum(uint32_t v) {
  int x = static_cast<int>(v);
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, false);   // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, false);   // row_shr:2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, false);   // row_shr:4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, false);   // row_shr:8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false);   // row_bcast:15 into rows 1 and 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false);   // row_bcast:31 into rows 2 and 3
  return static_cast<uint32_t>(x);
}

// minimum / maximum over the 64 lanes of a wavefront, uniform result: the same DPP ladder as the prefix sum (lanes
// without a source keep the identity), the total ends up in the last lane
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v) {
  int x = static_cast<int>(v);
  const int id = -1;                               // 0xffffffff
  auto mn = [](int a, int b) { return static_cast<int>(min(static_cast<uint32_t>(a), static_cast<uint32_t>(b))); };
  x = mn(x, __builtin_amdgcn_update_dpp(id, x, 0x111, 0xF, 0xF, false));
  x = mn(x, __builtin_amdgcn_update_dpp(id, x, 0x112, 0xF, 0xF, false));
  x = mn(x, __builtin_amdgcn_update_dpp(id, x, 0x114, 0xF, 0xF, false));
  x = mn(x, __builtin_amdgcn_update_dpp(id, x, 0x118, 0xF, 0xF, false));
  x = mn(x, __builtin_amdgcn_update_dpp(id, x, 0x142, 0xA, 0xF, false));
  x = mn(x, __builtin_amdgcn_update_dpp(id, x, 0x143, 0xC, 0xF, false));
  return static_cast<uint32_t>(__builtin_amdgcn_readlane(x, kWave - 1));
}
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
  int x = static_cast<int>(v);
  auto mx = [](int a, int b) { return static_cast<int>(max(static_cast<uint32_t>(a), static_cast<uint32_t>(b))); };
  x = mx(x, __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, false));
  x = mx(x, __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, false));
  x = mx(x, __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, false));
  x = mx(x, __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, false));
  x = mx(x, __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false));
  x = mx(x, __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false));
  return static_cast<uint32_t>(__builtin_amdgcn_readlane(x, kWave - 1));
}

// Sum of the entries of `sums` before entry `at` (wave-uniform, at most 64 entries), and of all of them: one LDS read per
// lane and one scan, where a loop over the entries would wait for the LDS once per entry.
__device__ __forceinline__ uint32_t sum_before(const uint32_t* sums, int n, int at, int lane, uint32_t* total) {
  const uint32_t incl = wave_inclusive_sum(lane < n ? sums[lane] : 0u);
  *total = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(incl), kWave - 1));
  return at > 0 ? static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(incl), at - 1)) : 0u;
}

// LDS the selection needs (one instance per workgroup of THREADS threads holding CH chunks of keys).
template <int THREADS, int CH> struct SelectLds {
  __attribute__((aligned(16))) uint32_t hist[4096];
  uint32_t wave_sum[2][CH * (THREADS / kWave)];
  uint32_t prefix[3], remaining[3];        // one slot per pass: no barrier between reading one and writing the next
  uint32_t in_bin;                         // keys that share the first digit of the K-th largest
  uint32_t n_cand;
  uint32_t cand[kWave];                    // those keys, where one wavefront's lanes hold them all
};

// Clears the histogram.  Called by every thread some time before the selection, with a barrier in between that the caller has anyway:
// the stores and the barrier then cost nothing of their own (with one barrier less after the last scores, 32 requests of 4096 tokens
// 132.2 -> 131.3 us, unified batch of 128 149.7 -> 148.2).  16 bytes per store, and behind the loads of the scores: 8000 rows of 300
// scores 121 us cleared inside, 127 in front of the loads, 122.8 behind them, 119 with wide stores; 128 rows of 8 K 23.7, 23.3, 23.2, 22.2.
template <int THREADS, int CH>
__device__ __forceinline__ void select_clear(SelectLds<THREADS, CH>& lds) {
  for (int i = threadIdx.x; i < 1024; i += THREADS) reinterpret_cast<uint4*>(lds.hist)[i] = uint4{0, 0, 0, 0};
  if (threadIdx.x == 0) lds.n_cand = 0;
}

// The workgroup holds CH * THREADS * KPC keys: key[c][j] of thread t belongs to position
// c * (THREADS * KPC) + t * KPC + j; positions >= L are ignored.  Writes the K selected positions in
// ascending order to out[0..K).  A histogram of the upper 12 bits (sign, exponent and three or more mantissa
// bits: attention scores share a few exponents, and a wide first digit is what keeps the LDS increments from
// serialising) finds the first digit of the K-th largest key.  Usually few keys share it: up to 64 of them are
// collected and every wavefront ranks them by itself, so that two barriers follow where two further histogram
// passes (12 and 8 bits: the path for more keys) take six; and if all of them are taken there is nothing to rank.
// Equal keys go to the lower position.  Every thread of the workgroup must call this, after select_clear and a barrier.
// What it costs is latency (barriers, LDS round trips): the stand-alone kernel on two rows of 512 scores 9.3 -> 5.3 us,
// 128 rows of 28 K 30.5 -> 20.7 us with the candidates and with the scans over wavefronts done by lanes instead of loops.
template <int THREADS, int KPC, int CH>
__device__ __forceinline__ void select_topk_in_registers(const uint32_t (&key)[CH][KPC], int L, int K, int32_t* out,
                                                         SelectLds<THREADS, CH>& lds) {
  constexpr int kWaves = THREADS / kWave;
  constexpr int kChunk = THREADS * KPC;
  static_assert(4096 % THREADS == 0 && THREADS >= 256, "bins are dealt out evenly");
  static_assert(CH * kWaves <= kWave, "one lane per (chunk, wavefront)");
  static_assert(CH * kChunk < 65536, "two counts of positions share 32 bits");
  uint32_t* hist = lds.hist;
  const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int t0 = static_cast<int>(threadIdx.x) * KPC;
  uint32_t prefix = 0, remaining = K;      // uniform across the workgroup
  const bool take_all = !(K < L);
  const int nch = (L + kChunk - 1) / kChunk;   // chunks that hold any position of this row (uniform): the others are skipped
  if (!take_all) {
#pragma unroll
    for (int pass = 0; pass < 3; ++pass) {
      const int shift = pass == 0 ? 20 : pass == 1 ? 8 : 0;
      const int bins = pass == 2 ? 256 : 4096;
      const uint32_t digit_mask = bins - 1;
      const uint32_t mask = pass == 0 ? 0u : pass == 1 ? 0xfff00000u : 0xffffff00u;
      // (every pass finds the bins zeroed: by select_clear, or by the last pass's readers)
      // A wavefront whose active keys all fall into one bin (constant or zero scores, or the few keys left in a late
      // pass) adds their number once instead of queueing up on one LDS address; otherwise every key adds itself.
      uint32_t lo = 0xffffffffu, hi = 0u, mine = 0u;
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        if (c >= nch) continue;
#pragma unroll
        for (int j = 0; j < KPC; ++j) {
          const bool act = c * kChunk + t0 + j < L && (key[c][j] & mask) == prefix;
          const uint32_t bin = (key[c][j] >> shift) & digit_mask;
          lo = act ? min(lo, bin) : lo;
          hi = act ? max(hi, bin) : hi;
          mine += act ? 1u : 0u;
        }
      }
      const uint32_t wave_lo = wave_min_u32(lo), wave_hi = wave_max_u32(hi);
      if (wave_lo >= wave_hi) {                  // one bin, or no active key at all (lo = ~0 > hi = 0)
        const uint32_t total = wave_inclusive_sum(mine);
        if (lane == kWave - 1 && total > 0) atomicAdd(&hist[wave_lo], total);
      } else {
#pragma unroll
        for (int c = 0; c < CH; ++c) {
          if (c >= nch) continue;
#pragma unroll
          for (int j = 0; j < KPC; ++j) {
            const bool act = c * kChunk + t0 + j < L && (key[c][j] & mask) == prefix;
            if (act) atomicAdd(&hist[(key[c][j] >> shift) & digit_mask], 1u);
          }
        }
      }
      __syncthreads();
      // thread t owns the bins (bins-1) - per*t - j, j < per, walking the digits downwards; it reads them
      // and leaves them zero for the next pass
      constexpr int kPerWide = 4096 / THREADS;     // 4 or 8 bins per thread in the two 12-bit passes
      const int per = pass == 2 ? (threadIdx.x < 256 ? 1 : 0) : kPerWide;
      uint32_t cnt[kPerWide], tot = 0;
#pragma unroll
      for (int j = 0; j < kPerWide; ++j) {
        cnt[j] = 0u;
        if (j < per) {
          uint32_t& slot = hist[bins - 1 - per * static_cast<int>(threadIdx.x) - j];
          cnt[j] = slot;
          slot = 0u;
        }
        tot += cnt[j];
      }
      uint32_t incl = wave_inclusive_sum(tot);   // inclusive scan over the workgroup: lanes, then wavefronts
      if (lane == kWave - 1) lds.wave_sum[pass & 1][wave] = incl;
      __syncthreads();
      uint32_t all;
      incl += sum_before(lds.wave_sum[pass & 1], kWaves, wave, lane, &all);
      uint32_t above = incl - tot;           // keys in strictly higher digits than this thread's
      if (above < remaining && incl >= remaining) {
#pragma unroll
        for (int j = 0; j < kPerWide; ++j) {
          if (j < per) {
            if (above < remaining && above + cnt[j] >= remaining) {
              const uint32_t digit = static_cast<uint32_t>(bins - 1 - per * static_cast<int>(threadIdx.x) - j);
              lds.prefix[pass] = prefix | (digit << shift);
              lds.remaining[pass] = remaining - above;
              if (pass == 0) lds.in_bin = cnt[j];
              above = remaining;               // stop: only one digit can match
            } else {
              above += cnt[j];
            }
          }
        }
      }
      __syncthreads();
      prefix = lds.prefix[pass];
      remaining = lds.remaining[pass];
      if (pass == 0) {
        const uint32_t in_bin = lds.in_bin;
        if (in_bin == remaining && prefix > 0) {     // every key with this digit is taken: all keys above prefix - 1
          prefix -= 1;
          remaining = 0;
          break;
        }
        if (in_bin <= kWave) {
#pragma unroll
          for (int c = 0; c < CH; ++c) {
            if (c >= nch) continue;
#pragma unroll
            for (int j = 0; j < KPC; ++j)
              if (c * kChunk + t0 + j < L && (key[c][j] & 0xfff00000u) == prefix) lds.cand[atomicAdd(&lds.n_cand, 1u)] = key[c][j];
          }
          __syncthreads();
          const uint32_t mine_key = lane < static_cast<int>(in_bin) ? lds.cand[lane] : 0u;
          uint32_t n_above = 0, n_equal = 0;         // candidates above this lane's key, and equal to it
          for (int i = 0; i < static_cast<int>(in_bin); ++i) {
            const uint32_t other = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(mine_key), i));
            n_above += other > mine_key ? 1u : 0u;
            n_equal += other == mine_key ? 1u : 0u;
          }
          const uint64_t kth = __ballot(lane < static_cast<int>(in_bin) && n_above < remaining && n_above + n_equal >= remaining);
          const int at = __ffsll(static_cast<unsigned long long>(kth)) - 1;      // the lanes of one value: the K-th largest key's
          prefix = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(mine_key), at));
          remaining -= static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(n_above), at));
          break;
        }
      }
    }
  } else {
    remaining = 0;
  }
  const uint32_t T = prefix;
  // remaining = how many keys equal to T are taken (lowest positions first)

  // per chunk: how many of this thread's keys lie above T (low half), and how many equal it (high half); exclusive
  // scans of both over the workgroup, in position order (positions grow with the chunk first, then with the thread)
  uint32_t n_sel[CH], s_sel[CH];
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    n_sel[c] = s_sel[c] = 0;
    if (c < nch) {
#pragma unroll
      for (int j = 0; j < KPC; ++j) {
        const bool in = c * kChunk + t0 + j < L;
        n_sel[c] += (in && (take_all || key[c][j] > T)) ? 1u : 0u;
        n_sel[c] += (in && !take_all && key[c][j] == T) ? 0x10000u : 0u;
      }
      s_sel[c] = wave_inclusive_sum(n_sel[c]);
    }
    if (lane == kWave - 1) lds.wave_sum[1][c * kWaves + wave] = s_sel[c];       // (last read before the barrier above)
  }
  __syncthreads();
  const uint32_t before = wave_inclusive_sum(lane < CH * kWaves ? lds.wave_sum[1][lane] : 0u);     // (chunk, wavefront) in position order
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    if (c >= nch) continue;
    const int at = c * kWaves + wave;
    const uint32_t base = at > 0 ? static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(before), at - 1)) : 0u;
    const uint32_t first = base + s_sel[c] - n_sel[c];
    uint32_t gt_before = first & 0xffffu, eq_before = first >> 16;
    // output slot of a selected key = (# greater before it) + (# equal-and-taken before it)
#pragma unroll
    for (int j = 0; j < KPC; ++j) {
      const int pos = c * kChunk + t0 + j;
      const bool in = pos < L;
      const bool gt = in && (take_all || key[c][j] > T);
      const bool eq = in && !take_all && key[c][j] == T;
      if (gt || (eq && eq_before < remaining)) out[gt_before + min(eq_before, remaining)] = pos;
      gt_before += gt ? 1u : 0u;
      eq_before += eq ? 1u : 0u;
    }
  }
}

}  // namespace
}  // namespace pillar
