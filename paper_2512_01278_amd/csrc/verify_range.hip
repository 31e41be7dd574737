// Verification attention with the score statistic (paper Section 4.1) as
// streaming passes over an evenly divided token range.
//
// The probability of a token needs the row's log-sum-exp over the WHOLE
// context, which is known only after the last token.  Two ways round it live
// here; kernel boundaries are the only synchronisation in both.
//
// Default, K read once:
//   single pass       S^T = K Q^T and O^T = V^T P^T on the matrix cores the
//                     flash-decoding way (running max and sum per row, one
//                     unnormalised (m, l, O) partial per segment); the
//                     exponentials e = exp2(s - m_tile) are left behind as
//                     16-bit values (verify_flash_team with four wavefronts
//                     per range, up to 32 rows, 48 with fp8;
//                     verify_flash_pair with two for more; mixed_flash_team
//                     and mixed_flash_pair with the draft step of other
//                     requests in the same grid, paper Section 4.2)
//   finish            per (request, KV head), one launch (verify_finish):
//                     log-sum-exp per row from the segments, O of pairs cut
//                     into several segments, scores = mean over rows of
//                     e * exp2(m_tile - lse) read back from the stash, and
//                     Top-K of those scores while they are still on the chip
//                     (long rows with few pairs: several workgroups per pair,
//                     then verify_select_rows)
//
// Variant with fp32 probabilities, K read twice (PILLAR_FLAG_EXACT_SCORES):
//   pass 1 (K only)   running (max, sum) per row -> (m, l) per row and segment
//   combine           as above
//   pass 2 (K and V)  p = exp2(s - lse) is the exact probability: the score is
//                     written directly, and O needs no running maximum;
//                     segment partials of O add linearly
//   merge             O = sum of the partials
//
// Work division.  The unit of work is a tile of 32 tokens of one (request, KV
// head) pair; all units are laid out pair-major (request, head, tile) and the
// T units are cut into N equal contiguous ranges, one per workgroup, N being
// the number of workgroups the chip holds at once.  Every workgroup therefore
// streams the same number of bytes and the grid drains all at once; a fixed
// slice size instead leaves the last round of workgroups on a half-empty chip
// (measured: a third of the pass-2 time at batch 128).  A range crosses pair
// boundaries; the stretch of one pair inside one range is a segment, and the
// segment of pair p in range w owns partial-result slot p + w (distinct
// segments have distinct sums because both indices grow along the layout).
// The plan (unit prefix per request, order of the pairs for the finish kernel)
// is a small kernel of its own (range_plan), or, for the single pass with up to
// 1024 requests, worked out by the wavefronts of the pass themselves (wave_plan).
#include <type_traits>

#include "host_rules.hpp"
#include "launch.hpp"
#include "mfma_tile.hpp"
#include "topk_core.hpp"
#include "verify_stream.hpp"
#include "decode_span.hpp"

namespace pillar {
namespace {

constexpr int kThreads = 64;                   // one wavefront per workgroup
constexpr int kWindowPages = 64;               // page ids held per register: one per lane
constexpr int kFinishMaxTokens = 32768;        // longest row whose Top-K the finish kernel selects itself

struct RangeWs {
  int32_t* ctrl;        // [0] total units T  [1] 0: equal ranges; else a range is a piece of one pair, at most 2^(ctrl[1] - 1) tiles
  int32_t* ureq;        // [B+1] first unit of request b (its heads follow each other)
  int32_t* order;       // [pairs] (request, head) pairs in the order the finish kernel takes them: longest rows first.  Null for a finish
                        // kernel of one workgroup per pair that all run at once; those that share pairs, and verify_select_rows, read it
  float* scratch_scores;  // [pairs][scratch_stride] statistic of the split finish kernel when the caller wants none
  int64_t scratch_stride;
  float* part_m;        // [pairs + N][rows_pad]  log2 domain
  float* part_l;        // [pairs + N][rows_pad]
  float* part_o;        // [pairs + N][R][128]
  float* lse2;          // [pairs][rows_pad]      log2 domain
  uint8_t* stash;       // single-pass variant: [units][tile lanes][16 bytes]
  float* m_ref;         //                      [units][rows_pad] running maximum the stash of a tile refers to (-inf: the row sees nothing yet)
  const int32_t* spec_lens;   // [B] speculative length of each request, or null: all use the call's k
  int32_t rows_pad;     // 16 * row blocks
  int32_t n_ranges;     // N
  int32_t plan_in_wave; // ctrl / ureq / order are not there yet: the wavefronts of the single pass work them out (wave_plan)
};

__host__ __device__ inline int tiles_of_len(int len) { return (len + kTileTokens - 1) / kTileTokens; }

// query positions of request b: all n_q slots, or as many as the request speculates
__device__ __forceinline__ int queries_of(const KvView& kv, const RangeWs& ws, int b, int n_q) {
  return ws.spec_lens ? min(ws.spec_lens[request_of(kv, b)] + 1, n_q) : n_q;
}

// Ranges in use: all that the chip holds at once, but none shorter than kMinTiles tiles.  A segment more to merge costs the
// finish kernel little, a segment more in a range a workgroup one after the other: pass + finish at one request of 2100
// tokens 11.3 + 15.2 us with 2 tiles, 13.2 + 14.2 with 4, 14.8 + 12.8 with 8; 24 requests of 5 to 3000 tokens 17.0 + 16.2,
// 23.0 + 14.2, 39.6 + 12.8.  (With 1, every tile a segment: 12.4 + 20.4 and 14.3 + 20.4 with a range per wavefront.  Both of these batches
// are cut into pieces now, below.  Left to this rule are batches of more short pairs than there are ranges, those of more than 1024
// requests, and the exact variant.)
constexpr int kMinTiles = 2;
__device__ __forceinline__ int ranges_used(const RangeWs& ws, int total) { return max(1, min(ws.n_ranges, total / kMinTiles)); }

// first unit of range w, and the range a unit falls in
__device__ __forceinline__ int range_begin(int w, int total, int n) { return static_cast<int>(static_cast<int64_t>(w) * total / n); }
__device__ __forceinline__ int range_of(int unit, int total, int n) {
  return static_cast<int>(((static_cast<int64_t>(unit) + 1) * n - 1) / total);
}

// Small batches: pieces of one pair instead of equal ranges.  A range of a few tiles that crosses from pair to pair takes as long as its
// stretches together (each a chain of loads and a merge), and the grid as long as that.  So a batch whose pairs make no more pieces
// of at most 4, 8, 16 or 32 tiles than there are ranges is cut that way, into the shortest such pieces, one per range: a team has a tile per
// wavefront in the shortest, and shorter ones would only leave more partials.  Equal ranges / pieces, pass + finish: 24 requests of 5-3000
// tokens, 4 heads 15.5 + 14.9 / 11.4 + 12.4 us, one of 2100 11.0 + 15.2 / 10.0 + 12.5, 2 of 6-8 K 43.3 / 36.8 in all, fp8 with 40
// rows 8 of 1-4 K 42.7 / 38.1 and 12 of 3-7 K 61.6 / 57.7, 24 of 10-3000 with 64 rows 47.6 / 35.0.
// A piece may be longer than an equal range by what a boundary costs, some 8 tiles: 64 pairs of 17 x 256 tokens (pieces of 32 tiles,
// ranges of 17) 48.8 / 50.5 us, of 14 x 256 (16 against 14) 43.6 / 37.9.  The pass with two wavefronts per range goes through a tile with
// both, so that a longer range costs it more than a boundary: pieces of 2 and of 4 tiles only (128 pairs, 36 rows, pieces of 16 against
// ranges of 9 62.5 / 73.7, 64 rows, of 8 against 6 49.5 / 55.9).  (These with pieces of 2^n tiles and a rest.)
// Pieces of 2 for that pass, up to half as many as there are ranges, beyond which their partials cost as much.  8 heads, equal ranges / pieces
// of 4 / of 2: one request of 100 tokens, 64 rows 19.4 / 20.5 / 17.6 us, of 1000 33.2 / 22.4 / 20.4, of 2000 47.1 / 25.5 / 22.5; 4 of 256
// 22.0 / 21.8 / 19.6; 8 of 270-300 with 36 rows 24.2 / 21.7 / 20.1, of 480-720 (640 pieces) 29.1 / 23.2 / 24.1.
constexpr int kMinTeamPiece = 2, kMaxTeamPiece = 5, kMinPairPiece = 1, kMaxPairPiece = 2, kPieceSlack = 8;

// Segments of a pair that begins at unit u0, and the slot of the first: pair + range, or that of its first piece.
struct PairSegs { int slot0, n; };
__device__ __forceinline__ PairSegs segs_of_pair(const RangeWs& ws, int total, int cut, int pair, int u0, int tiles) {
  if (cut > 0) return PairSegs{pair + first_slot(u0, cut - 1), pieces_of(tiles, cut - 1)};
  const int n = ranges_used(ws, total), w0 = range_of(u0, total, n);
  return PairSegs{pair + w0, range_of(u0 + tiles - 1, total, n) - w0 + 1};
}

// ---------------------------------------------------------------- plan ------
// Unit prefix per request, and the order in which the finish kernel takes the (request, head) pairs:
// longest requests first, so that the workgroups still running when the grid drains are short ones.
__global__ __launch_bounds__(1024) void range_plan(KvView kv, RangeWs ws) {
  __shared__ int32_t scan[1024];
  __shared__ int32_t carry;
  if (threadIdx.x == 0) carry = 0;
  __syncthreads();
  int first_len = 0;                           // length of request threadIdx.x (first pass), for the ranking below
  for (int b0 = 0; b0 < kv.batch; b0 += 1024) {
    const int b = b0 + threadIdx.x;
    const int len_b = b < kv.batch ? kv.seq_lens[request_of(kv, b)] : 0;
    if (b0 == 0) first_len = len_b;
    const int mine = b < kv.batch ? tiles_of_len(len_b) * kv.num_kv_heads : 0;
    scan[threadIdx.x] = mine;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
      const int v = threadIdx.x >= o ? scan[threadIdx.x - o] : 0;
      __syncthreads();
      scan[threadIdx.x] += v;
      __syncthreads();
    }
    if (b < kv.batch) ws.ureq[b] = carry + scan[threadIdx.x] - mine;
    __syncthreads();
    if (threadIdx.x == 1023) carry += scan[1023];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    ws.ureq[kv.batch] = carry;
    ws.ctrl[0] = carry;
    ws.ctrl[1] = 0;
  }
  // rank of every request by length (ties by index); batches beyond one workgroup keep their own order
  if (kv.batch <= 1024) {
    __syncthreads();
    const int b = threadIdx.x;
    const int len = first_len;
    scan[threadIdx.x] = len;
    __syncthreads();
    if (b < kv.batch) {
      int rank = 0;
      for (int o = 0; o < kv.batch; ++o) {
        const int lo = scan[o];
        rank += (lo > len || (lo == len && o < b)) ? 1 : 0;
      }
      for (int g = 0; g < kv.num_kv_heads; ++g) ws.order[rank * kv.num_kv_heads + g] = b * kv.num_kv_heads + g;
    }
  } else {
    for (int i = threadIdx.x; i < kv.batch * kv.num_kv_heads; i += 1024) ws.order[i] = i;
  }
}

// ------------------------------------------------------------- helpers ------
// One stretch of one pair inside one range.
struct Segment {
  int b, g, L, tiles, tile0, tile1, pair, slot;   // b: slot of the request in this launch
  int rq;                                          // the request's id: index into everything the request owns
};

// request whose units contain `unit`: two rounds of 64-way search, the prefix table stays in L2
__device__ __forceinline__ int find_request(const RangeWs& ws, int batch, int unit, int lane) {
  int lo = 0, n = batch;                       // answer in [lo, lo + n)
  while (n > 1) {
    const int step = (n + kThreads - 1) / kThreads;
    const int probe = lo + min(lane * step, n - 1);
    const bool le = ws.ureq[probe] <= unit;    // true for a prefix of the lanes (lane 0 always)
    const int hits = __popcll(__ballot(le));
    const int first = lo + min((hits - 1) * step, n - 1);
    n = min(step, lo + n - first);
    lo = first;
  }
  return __builtin_amdgcn_readfirstlane(lo);
}

// page ids of the 64-page windows `win` and `win + 1` of a request: lane j holds page 64 * win + j
struct PageWin {
  int pg_a, pg_b, win;
};

__device__ __forceinline__ int load_window(const KvView& kv, int b, int win, int lane);

// Issues the loads of the tile at token tb (K rows into rk when WITH_K, V rows into rv when
// WITH_V) and reports the pages of its two 16-token halves.  Tiles are issued in ascending
// order, so the page window only ever moves forward; a 16-token group lies in one page whose
// id is wave-uniform, which makes the address a scalar base plus a 32-bit per-lane offset.
// Groups beyond the end of the sequence read the last page of the request: pages are whole, so
// the rows exist; the caller masks them.
template <bool FP8, bool WITH_K, bool WITH_V>
__device__ __forceinline__ void issue_tile(const KvView& kv, const Segment& sg, int tb, PageWin& pw, const LaneGeom<FP8>& geo,
                                           int lane, u32x4 (&rk)[TileRegs<FP8>::kLoads], u32x4 (&rv)[TileRegs<FP8>::kLoads],
                                           int (&pages)[2]) {
  constexpr int kLoads = TileRegs<FP8>::kLoads;
  constexpr int kPerGroup = kLoads / 2;
  const int esz = FP8 ? 1 : 2;
  const int last_page = (sg.L - 1) >> kv.page_shift;
  // both 16-token groups of a tile lie in the same 64-page window (pages hold >= 16 tokens and a tile starts
  // at a multiple of 32 tokens), so the window moves at most once per tile, before any row load is issued
  if (min(tb >> kv.page_shift, last_page) / kWindowPages > pw.win) {          // wave-uniform
    pw.pg_a = pw.pg_b;
    pw.win += 1;
    pw.pg_b = load_window(kv, sg.b, pw.win + 1, lane);
  }
#pragma unroll
  for (int grp = 0; grp < 2; ++grp) {
    const int tok0 = tb + 16 * grp;
    const int lp = min(tok0 >> kv.page_shift, last_page);
    const int page = __builtin_amdgcn_readlane(pw.pg_a, lp - pw.win * kWindowPages);
    pages[grp] = page;
    const int64_t base = (static_cast<int64_t>(page) * kv.stride_page + static_cast<int64_t>(sg.g) * kv.stride_head +
                          static_cast<int64_t>(tok0 & (kv.page_size - 1)) * kv.stride_slot) * esz;
    const char* gk = static_cast<const char*>(kv.k_pool) + base;
    const char* gv = static_cast<const char*>(kv.v_pool) + base;
#pragma unroll
    for (int u = 0; u < kPerGroup; ++u) {
      const int64_t step = u * geo.row_step;
      if constexpr (WITH_K) rk[grp * kPerGroup + u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(gk + step + geo.lane_off));
      if constexpr (WITH_V) rv[grp * kPerGroup + u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(gv + step + geo.lane_off));
    }
  }
}

// fp8: dequantisation scales of the two 16-token halves of a tile
__device__ __forceinline__ void half_scales(const KvView& kv, int g, const int (&pages)[2], const float* table, float (&sc)[2]) {
#pragma unroll
  for (int sub = 0; sub < 2; ++sub) sc[sub] = table[static_cast<int64_t>(pages[sub]) * kv.num_kv_heads + g];
}

template <int RB>
__device__ __forceinline__ void load_q_regs(const KvView& kv, const uint16_t* q, int n_q, int G, int R, const Segment& sg,
                                            bf16x8 (&qf)[RB][4], int lane) {
  const int n = lane & 15, g4 = lane >> 4;
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const int r = 16 * rb + n;
    const int i = r / G, hg = r - i * G;
    const uint16_t* row = q + ((static_cast<int64_t>(sg.rq) * n_q + i) * kv.num_q_heads + sg.g * G + hg) * kHeadDim;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      u32x4 v = {0u, 0u, 0u, 0u};
      if (r < R) v = *reinterpret_cast<const u32x4*>(row + 32 * s + 8 * g4);
      qf[rb][s] = as_bf16x8(v);
    }
  }
}

// A tile on its way from HBM to a register set: which segment it belongs to and where it starts.
struct Flight {
  Segment sg;
  int tb;            // first token of the tile
  int pages[2];      // pages of its two 16-token halves
  float ks[2], vs[2];  // fp8: dequantisation scales of those pages, fetched along with the rows (a load at the
                     // tile's turn would keep a round trip to memory in every tile)
  bool valid;
};

template <bool FP8>
__device__ __forceinline__ void fetch_scales(const KvView& kv, Flight& f) {
  f.ks[0] = f.ks[1] = f.vs[0] = f.vs[1] = 1.f;
  if constexpr (FP8) {
    half_scales(kv, f.sg.g, f.pages, kv.k_scale, f.ks);
    half_scales(kv, f.sg.g, f.pages, kv.v_scale, f.vs);
  }
}

// Issue side of the tile stream of one range.  The stream runs ahead of the arithmetic by the
// tiles in flight and crosses pair boundaries without draining: when it enters a pair it already
// holds the page ids of the pair after it (they were fetched one pair earlier).
struct Cursor {
  int unit, end, slot;  // next unit to issue, end of the range, slot of a segment less its pair
  Segment sg;        // the segment that unit belongs to
  int tile;          // next tile of sg
  PageWin pw;
  int pg_next;       // page window 0 of the request of the following pair
  int len_next;      // sequence length of that request (per-lane copy)
  bool live;
};

__device__ __forceinline__ int load_window(const KvView& kv, int b, int win, int lane) {
  // entries past the last page of the request are never used as addresses (issue_tile clamps), so
  // it is enough to stay inside the table row
  return kv.block_table[static_cast<int64_t>(request_of(kv, b)) * kv.block_table_stride + min(win * kWindowPages + lane, kv.block_table_stride - 1)];
}

__device__ __forceinline__ void prefetch_following(const KvView& kv, Cursor& c, int lane) {
  int nb = c.sg.b + (c.sg.g + 1 == kv.num_kv_heads ? 1 : 0);
  nb = min(nb, kv.batch - 1);                  // past the last request nothing of this is used
  c.len_next = kv.seq_lens[request_of(kv, nb)];
  c.pg_next = load_window(kv, nb, 0, lane);
}

__device__ __forceinline__ Segment uniform(const Segment& s) {
  Segment u;
  u.b = __builtin_amdgcn_readfirstlane(s.b);
  u.g = __builtin_amdgcn_readfirstlane(s.g);
  u.L = __builtin_amdgcn_readfirstlane(s.L);
  u.tiles = __builtin_amdgcn_readfirstlane(s.tiles);
  u.tile0 = __builtin_amdgcn_readfirstlane(s.tile0);
  u.tile1 = __builtin_amdgcn_readfirstlane(s.tile1);
  u.pair = __builtin_amdgcn_readfirstlane(s.pair);
  u.slot = __builtin_amdgcn_readfirstlane(s.slot);
  u.rq = __builtin_amdgcn_readfirstlane(s.rq);
  return u;
}

// The plan without a launch of its own, for batches of up to 64 * kPlanRegs requests: every wavefront of the
// single pass reads all lengths (lane l, register j: request 64 j + l) and scans them into the unit prefix, which
// costs one round trip to memory where reading a finished plan costs three dependent ones.
constexpr int kPlanRegs = 16;
template <int REGS> struct WavePlan {
  int len[REGS];
  int first[REGS];        // units before the request
  int total;
};

template <int REGS>
__device__ __forceinline__ WavePlan<REGS> wave_plan(const KvView& kv, int lane) {
  WavePlan<REGS> p;
#pragma unroll
  for (int j = 0; j < REGS; ++j) {
    p.len[j] = 0;
    if (kWave * j < kv.batch) {                // wave-uniform
      const int b = kWave * j + lane;
      if (b < kv.batch) p.len[j] = kv.seq_lens[request_of(kv, b)];
    }
  }
  int carry = 0;
#pragma unroll
  for (int j = 0; j < REGS; ++j) {
    p.first[j] = carry;
    if (kWave * j < kv.batch) {
      const int mine = tiles_of_len(p.len[j]) * kv.num_kv_heads;         // 0 beyond the batch
      const int incl = static_cast<int>(wave_inclusive_sum(static_cast<uint32_t>(mine)));
      p.first[j] = carry + incl - mine;
      carry += __builtin_amdgcn_readlane(incl, kWave - 1);
    }
  }
  p.total = carry;
  return p;
}

// value of register set v for request b (wave-uniform)
template <int REGS>
__device__ __forceinline__ int plan_get(const int (&v)[REGS], int b) {
  int r = 0;
#pragma unroll
  for (int j = 0; j < REGS; ++j)
    if (j == (b >> 6)) r = __builtin_amdgcn_readlane(v[j], b & (kWave - 1));
  return r;
}

// What range_plan leaves in memory for the kernels after the pass, written by the pass itself: wavefront w ranks
// requests w, w + N, ... by length (the order of the finish kernel: longest first, ties by index), wavefront 0
// also writes the prefix.
template <int REGS>
__device__ __forceinline__ void publish_plan(const KvView& kv, const RangeWs& ws, const WavePlan<REGS>& p, int cut, int w, int lane) {
  for (int r = w; r < kv.batch; r += ws.n_ranges) {
    const int len_r = plan_get(p.len, r);
    int rank = 0;
#pragma unroll
    for (int j = 0; j < REGS; ++j) {
      if (kWave * j < kv.batch) {
        const int b = kWave * j + lane;
        const bool ahead = b < kv.batch && (p.len[j] > len_r || (p.len[j] == len_r && b < r));
        rank += __popcll(__ballot(ahead));
      }
    }
    for (int g = lane; g < kv.num_kv_heads; g += kWave) ws.order[rank * kv.num_kv_heads + g] = r * kv.num_kv_heads + g;
  }
  if (w == 0) {
#pragma unroll
    for (int j = 0; j < REGS; ++j) {
      const int b = kWave * j + lane;
      if (b < kv.batch) ws.ureq[b] = p.first[j];
    }
    if (lane == 0) {
      ws.ureq[kv.batch] = p.total;
      ws.ctrl[0] = p.total;
      ws.ctrl[1] = cut;
    }
  }
}

// Where a range begins: its units and its first segment.  `publish`: this wavefront also writes its share of the plan to
// memory (one of those that share a range).
struct RangeStart {
  int unit, end;
  int slot;                // partial slot of the first segment, less its pair
  Segment sg;
  bool live;
};

// a / b, both below 2^22 (a piece has no more than 32 tiles, a range is no more than one), by a reciprocal of b that divisions share: at most one
// off before it is set right.
__device__ __forceinline__ int div_near(int a, int b, float rcp_b) {
  const int q = static_cast<int>(static_cast<float>(a) * rcp_b), r = a - q * b;
  return __builtin_amdgcn_readfirstlane(q + (r >= b) - (r < 0));
}

// The shortest pieces, of at most 2^MIN to 2^MAX tiles, with which the batch makes no more of them than there are ranges (log2 of their tiles
// plus one), or 0: equal ranges.  (MIN and MAX are constants and the loop stays one: what every workgroup has to fetch of code counts in small
// calls, with bounds in the arguments 24 requests of 5-3000 tokens 20.75 us instead of 20.6.)
template <int REGS, int MIN, int MAX>
__device__ __forceinline__ int plan_pieces(const KvView& kv, const RangeWs& ws, const WavePlan<REGS>& p, int lane) {
#pragma unroll 1
  for (int shift = MIN; shift <= MAX; ++shift) {
    const int most = shift == kMinPairPiece ? ws.n_ranges / 2 : ws.n_ranges;
    if (p.total > (most << shift)) continue;                           // too many whatever the lengths are
    if (shift > MIN && (ws.n_ranges << shift) > p.total + kPieceSlack * ws.n_ranges) return 0;
    int mine = 0;
#pragma unroll
    for (int j = 0; j < REGS; ++j) mine += pieces_of(tiles_of_len(p.len[j]), shift);         // 0 beyond the batch
    const int pieces = __builtin_amdgcn_readlane(static_cast<int>(wave_inclusive_sum(static_cast<uint32_t>(mine))), kWave - 1);
    if (pieces * kv.num_kv_heads <= most) return shift + 1;
  }
  return 0;
}

// The range's units and, if it has any, the request it begins in and that request's first unit, from lengths in registers.  Batches of up
// to 128 have a copy with two registers: stepping over the parts of the other fourteen, in every scan and every look-up, is
// some 500 instructions in a row, 1 us of each pass (one request of 2100 tokens, verification and draft, 30.4 -> 29.8 us, 24 of 5 to
// 3000 31.7 -> 30.8, 128 of 1-8 K 516.8 -> 514.5).
template <int REGS, int MIN, int MAX>
__device__ __forceinline__ void plan_range(const KvView& kv, const RangeWs& ws, int w, int lane, bool publish, RangeStart& c, int& first_unit) {
  const WavePlan<REGS> p = wave_plan<REGS>(kv, lane);
  const int cut = plan_pieces<REGS, MIN, MAX>(kv, ws, p, lane);
  if (publish) publish_plan(kv, ws, p, cut, w, lane);
  if (cut > 0) {
    const int shift = cut - 1;
    int carry = 0, upto = 0, before[REGS];                   // pieces before a request; requests that begin at or before piece w
#pragma unroll
    for (int j = 0; j < REGS; ++j) {
      before[j] = carry;
      if (kWave * j < kv.batch) {
        const int mine = pieces_of(tiles_of_len(p.len[j]), shift) * kv.num_kv_heads;
        const int incl = static_cast<int>(wave_inclusive_sum(static_cast<uint32_t>(mine)));
        before[j] = carry + incl - mine;
        carry += __builtin_amdgcn_readlane(incl, kWave - 1);
        upto += __popcll(__ballot(kWave * j + lane < kv.batch && before[j] <= w));
      }
    }
    c.live = w < carry;
    if (!c.live) return;
    c.sg.b = upto - 1;
    c.sg.L = plan_get(p.len, c.sg.b);
    first_unit = plan_get(p.first, c.sg.b);
    const int tiles = tiles_of_len(c.sg.L), per_head = pieces_of(tiles, shift);
    const float rcp = __builtin_amdgcn_rcpf(static_cast<float>(per_head));       // (whole divisions: 24 requests of 5-3000 tokens 20.75 us, 20.6 so)
    const int least = div_near(tiles, per_head, rcp);
    const int rel = w - plan_get(before, c.sg.b), head = div_near(rel, per_head, rcp), piece = rel - head * per_head, u0 = first_unit + head * tiles;
    c.unit = u0 + piece_begin(tiles, per_head, least, piece);
    c.end = u0 + piece_begin(tiles, per_head, least, piece + 1);
    c.slot = first_slot(u0, shift) + piece;
    return;
  }
  c.slot = w;
  const int n = ranges_used(ws, p.total);
  c.unit = range_begin(w, p.total, n);
  c.end = range_begin(w + 1, p.total, n);
  c.live = w < n && c.unit < c.end;            // (a batch of empty contexts has one range of nothing)
  if (!c.live) return;
  int upto = 0;                                // requests that begin at or before the unit
#pragma unroll
  for (int j = 0; j < REGS; ++j) {
    if (kWave * j < kv.batch) upto += __popcll(__ballot(kWave * j + lane < kv.batch && p.first[j] <= c.unit));
  }
  c.sg.b = upto - 1;
  c.sg.L = plan_get(p.len, c.sg.b);
  first_unit = plan_get(p.first, c.sg.b);
}

template <int MIN, int MAX>
__device__ __forceinline__ RangeStart open_range(const KvView& kv, const RangeWs& ws, int w, int lane, bool publish) {
  RangeStart c;
  c.sg = Segment{};
  c.slot = w;
  int first_unit = 0;                          // of the request the range begins in
  if (ws.plan_in_wave) {                       // the same for the whole grid
    if (kv.batch <= 2 * kWave) plan_range<2, MIN, MAX>(kv, ws, w, lane, publish, c, first_unit);
    else plan_range<kPlanRegs, MIN, MAX>(kv, ws, w, lane, publish, c, first_unit);
    if (!c.live) return c;
  } else {
    const int total = ws.ctrl[0];
    const int n = ranges_used(ws, total);
    c.unit = range_begin(w, total, n);
    c.end = range_begin(w + 1, total, n);
    c.live = w < n && c.unit < c.end;
    if (!c.live) return c;
    c.sg.b = find_request(ws, kv.batch, c.unit, lane);
    c.sg.L = __builtin_amdgcn_readfirstlane(kv.seq_lens[request_of(kv, c.sg.b)]);
    first_unit = __builtin_amdgcn_readfirstlane(ws.ureq[c.sg.b]);
  }
  Segment& sg = c.sg;
  sg.rq = __builtin_amdgcn_readfirstlane(request_of(kv, sg.b));
  sg.tiles = tiles_of_len(sg.L);
  const int rel = c.unit - first_unit;
  sg.g = rel / sg.tiles;
  sg.tile0 = rel - sg.g * sg.tiles;
  sg.tile1 = min(sg.tiles, sg.tile0 + (c.end - c.unit));
  sg.pair = sg.b * kv.num_kv_heads + sg.g;
  sg.slot = sg.pair + c.slot;
  return c;
}

__device__ __forceinline__ Cursor open_cursor(const KvView& kv, const RangeWs& ws, int w, int lane) {
  const RangeStart start = open_range<kMinPairPiece, kMaxPairPiece>(kv, ws, w, lane, true);
  Cursor c;
  c.slot = start.slot;
  c.unit = start.unit;
  c.end = start.end;
  c.sg = start.sg;
  c.live = start.live;
  c.tile = c.sg.tile0;
  c.pw = PageWin{};
  c.pg_next = 0;
  c.len_next = 0;
  if (!c.live) return c;
  c.pw.win = ((c.sg.tile0 * kTileTokens) >> kv.page_shift) / kWindowPages;
  c.pw.pg_a = load_window(kv, c.sg.b, c.pw.win, lane);
  c.pw.pg_b = load_window(kv, c.sg.b, c.pw.win + 1, lane);
  prefetch_following(kv, c, lane);
  return c;
}

// Steps the cursor past the tile just issued; entering the next pair costs no wait (its pages were
// fetched one pair earlier).
__device__ __forceinline__ void advance_cursor(const KvView& kv, Cursor& c, int lane) {
  c.tile += 1;
  c.unit += 1;
  if (c.unit >= c.end) {
    c.live = false;
  } else if (c.tile == c.sg.tile1) {           // on to the next pair
    Segment sg = c.sg;
    sg.g += 1;
    if (sg.g == kv.num_kv_heads) {
      sg.g = 0;
      sg.b += 1;
    }
    sg.L = __builtin_amdgcn_readfirstlane(c.len_next);
    if (__builtin_expect(sg.L <= 0 && sg.b + 1 < kv.batch, 0)) {      // an empty context has no tile: on to one that has (units are left, so there is one)
      int b = sg.b;
      do sg.L = kv.seq_lens[request_of(kv, ++b)];
      while (sg.L <= 0 && b + 1 < kv.batch);
      sg.b = __builtin_amdgcn_readfirstlane(b);
      sg.L = __builtin_amdgcn_readfirstlane(sg.L);
      c.pg_next = load_window(kv, sg.b, 0, lane);
    }
    sg.tiles = tiles_of_len(sg.L);
    sg.tile0 = 0;
    sg.tile1 = min(sg.tiles, c.end - c.unit);
    sg.pair = sg.b * kv.num_kv_heads + sg.g;
    sg.slot = sg.pair + c.slot;
    sg.rq = request_of(kv, sg.b);
    c.sg = uniform(sg);
    c.tile = 0;
    c.pw.win = 0;
    c.pw.pg_a = c.pg_next;
    c.pw.pg_b = load_window(kv, c.sg.b, 1, lane);
    prefetch_following(kv, c, lane);
  }
}

// Issues the next tile of the stream into a register set and steps the cursor.
template <bool FP8, bool WITH_V>
__device__ __forceinline__ Flight issue_next(const KvView& kv, Cursor& c, const LaneGeom<FP8>& geo, int lane,
                                             u32x4 (&rk)[TileRegs<FP8>::kLoads], u32x4 (&rv)[TileRegs<FP8>::kLoads]) {
  Flight f;
  f.valid = c.live;
  f.sg = c.sg;
  f.tb = c.tile * kTileTokens;
  f.pages[0] = f.pages[1] = 0;
  f.ks[0] = f.ks[1] = f.vs[0] = f.vs[1] = 1.f;
  if (!c.live) return f;
  issue_tile<FP8, true, WITH_V>(kv, c.sg, f.tb, c.pw, geo, lane, rk, rv, f.pages);
  fetch_scales<FP8>(kv, f);
  advance_cursor(kv, c, lane);
  return f;
}

// ---------------------------------------------------------------- pass 1 ----
template <int RB, bool FP8>
__global__ __launch_bounds__(kThreads, 2) void verify_lse_range(KvView kv, const uint16_t* q, int n_q, RangeWs ws) {
  __shared__ __attribute__((aligned(16))) uint8_t s_tile[kKTileBytes];
  const int lane = threadIdx.x;
  const int n = lane & 15, g4 = lane >> 4;
  const int G = kv.num_q_heads / kv.num_kv_heads;
  const int R = n_q * G;
  const float c2 = kv.sm_scale * kLog2e;
  const LaneGeom<FP8> geo = lane_geom<FP8>(kv, lane);
  constexpr int kLoads = TileRegs<FP8>::kLoads;
  Cursor cur = open_cursor(kv, ws, blockIdx.x, lane);
  if (!cur.live) return;
  // K tiles travel two deep: even tiles through ra, odd tiles through rb_
  u32x4 ra[kLoads], rb_[kLoads], unused[kLoads];
  Flight fa = issue_next<FP8, false>(kv, cur, geo, lane, ra, unused);
  Flight fb = issue_next<FP8, false>(kv, cur, geo, lane, rb_, unused);
  Segment cs = fa.sg;
  bool started = false;
  bf16x8 qf[RB][4];
  float m_run[RB], l_run[RB];
  auto finish = [&]() {                        // the 4 token groups of a row -> the segment's (m, l)
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const float mx = max_over_groups(m_run[rb]);
      const float m_use = (mx == -INFINITY) ? 0.f : mx;
      float l = l_run[rb] * fast_exp2(m_run[rb] - m_use);
      l = sum_over_groups(l);
      if (g4 == 0) {
        ws.part_m[static_cast<int64_t>(cs.slot) * (RB * 16) + 16 * rb + n] = mx;
        ws.part_l[static_cast<int64_t>(cs.slot) * (RB * 16) + 16 * rb + n] = l;
      }
    }
  };
  auto tile = [&](Flight& f, u32x4 (&regs)[kLoads]) {
    if (!started || f.sg.slot != cs.slot) {    // wave-uniform: the stream has entered another pair
      if (started) finish();
      cs = f.sg;
      started = true;
      load_q_regs<RB>(kv, q, n_q, G, R, cs, qf, lane);
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) { m_run[rb] = -INFINITY; l_run[rb] = 0.f; }
    }
    const int tb = f.tb;
    rows_to_lds<FP8, false>(regs, s_tile, lane);
    const float ks[2] = {f.ks[0], f.ks[1]};
    f = issue_next<FP8, false>(kv, cur, geo, lane, regs, unused);
    f32x4 s[2][RB];
    tile_qk<RB>(s_tile, qf, s, lane);
    const bool edge = tb + kTileTokens > cs.L - n_q;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
#pragma unroll
      for (int sub = 0; sub < 2; ++sub) s[sub][rb] *= c2 * ks[sub];
      if (edge) {
        const int r = 16 * rb + n;
        const int last = cs.L - n_q + (r < R ? r / G : n_q - 1);
#pragma unroll
        for (int sub = 0; sub < 2; ++sub)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (tb + 16 * sub + 4 * g4 + i > last) s[sub][rb][i] = -INFINITY;
      }
      const float mx = fmaxf(fmaxf(fmaxf(s[0][rb][0], s[0][rb][1]), fmaxf(s[0][rb][2], s[0][rb][3])),
                             fmaxf(fmaxf(s[1][rb][0], s[1][rb][1]), fmaxf(s[1][rb][2], s[1][rb][3])));
      const float m_new = fmaxf(m_run[rb], mx);
      const float m_use = (m_new == -INFINITY) ? 0.f : m_new;
      float sum = 0.f;
#pragma unroll
      for (int i = 0; i < 4; ++i) sum += fast_exp2(s[0][rb][i] - m_use) + fast_exp2(s[1][rb][i] - m_use);
      l_run[rb] = l_run[rb] * fast_exp2(m_run[rb] - m_use) + sum;
      m_run[rb] = m_new;
    }
  };
  for (;;) {
    if (!fa.valid) break;
    tile(fa, ra);
    if (!fb.valid) break;
    tile(fb, rb_);
  }
  finish();
}

// ---------------------------------------------------------------- combine ---
// one thread per (pair, padded row)
__global__ __launch_bounds__(256) void verify_lse_combine_range(KvView kv, int n_q, RangeWs ws, float* lse_out) {
  const int rows = ws.rows_pad;
  const int idx = blockIdx.x * 256 + threadIdx.x;
  const int pairs = kv.batch * kv.num_kv_heads;
  if (idx >= pairs * rows) return;
  const int pair = idx / rows, row = idx - pair * rows;
  const int b = pair / kv.num_kv_heads, g = pair - b * kv.num_kv_heads;
  const int G = kv.num_q_heads / kv.num_kv_heads;
  const int total = ws.ctrl[0];
  const int rq = request_of(kv, b);
  const int tiles = tiles_of_len(kv.seq_lens[rq]);
  const int u0 = ws.ureq[b] + g * tiles;
  const int n_used = ranges_used(ws, total);
  const int w0 = tiles > 0 ? range_of(u0, total, n_used) : 0, w1 = tiles > 0 ? range_of(u0 + tiles - 1, total, n_used) : -1;   // (empty context: none)
  const float* pm = ws.part_m + static_cast<int64_t>(pair + w0) * rows + row;
  const float* pl = ws.part_l + static_cast<int64_t>(pair + w0) * rows + row;
  float m = -INFINITY, l = 0.f;
  for (int c = 0; c <= w1 - w0; ++c) {
    const float mc = pm[static_cast<int64_t>(c) * rows], lc = pl[static_cast<int64_t>(c) * rows];
    const float mn = fmaxf(m, mc);
    const float mu = (mn == -INFINITY) ? 0.f : mn;
    l = l * fast_exp2(m - mu) + lc * fast_exp2(mc - mu);
    m = mn;
  }
  // rows beyond the request's R, and rows that see no token at all (a context shorter than the request's
  // queries), get +inf so that their probabilities vanish where the log-sum-exp is applied
  const int Rb = queries_of(kv, ws, b, n_q) * G;
  const bool live = row < Rb && l > 0.f;
  const float v = live ? m + log2f(l) : INFINITY;
  ws.lse2[idx] = v;
  if (lse_out && row < Rb) {
    const int i = row / G, hg = row - i * G;
    lse_out[(static_cast<int64_t>(rq) * n_q + i) * kv.num_q_heads + g * G + hg] = live ? v * kLn2 : -INFINITY;
  }
}

// ---------------------------------------------------------------- pass 2 ----
template <int RB, bool FP8>
__global__ __launch_bounds__(kThreads, RB >= 3 ? 1 : 2) void verify_score_range(KvView kv, const uint16_t* q, int n_q, RangeWs ws,
                                                                                 uint16_t* out, float* scores, int64_t score_stride) {
  // one tile buffer: the K rows, then (once S^T is done) the V rows of the same tile
  __shared__ __attribute__((aligned(16))) uint8_t s_tile[kVTileBytes];
  __shared__ __attribute__((aligned(16))) uint8_t s_q[(RB * 16 + 1) * kKRow];
  const int lane = threadIdx.x;
  const int n = lane & 15, g4 = lane >> 4;
  const int G = kv.num_q_heads / kv.num_kv_heads;
  const int R = n_q * G;
  const float c2 = kv.sm_scale * kLog2e;
  const float inv_r = 1.0f / static_cast<float>(R);
  const LaneGeom<FP8> geo = lane_geom<FP8>(kv, lane);
  constexpr int kLoads = TileRegs<FP8>::kLoads;
  constexpr int kQIters = ((RB * 16 + 1) * 16 + kThreads - 1) / kThreads;
  Cursor cur = open_cursor(kv, ws, blockIdx.x, lane);
  if (!cur.live) return;
  u32x4 rk[kLoads], rv[kLoads];
  Flight f = issue_next<FP8, true>(kv, cur, geo, lane, rk, rv);
  Segment cs = f.sg;
  bool started = false;
  float lse2[RB];
  float* sdst = scores;
  f32x4 o[RB][8];
  auto finish = [&]() {                        // O of the segment: final when it is the whole pair, else a partial
    const bool whole = cs.tile0 == 0 && cs.tile1 == cs.tiles;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const int r = 16 * rb + n;
      if (r >= R) continue;
      if (whole) {
        const int i = r / G, hg = r - i * G;
        uint16_t* dst = out + ((static_cast<int64_t>(cs.rq) * n_q + i) * kv.num_q_heads + cs.g * G + hg) * kHeadDim;
#pragma unroll
        for (int db = 0; db < 8; ++db) {
          u32x2 pk;
          pk.x = pack2(o[rb][db][0], o[rb][db][1]);
          pk.y = pack2(o[rb][db][2], o[rb][db][3]);
          *reinterpret_cast<u32x2*>(dst + 16 * db + 4 * g4) = pk;
        }
      } else {
        float* dst = ws.part_o + (static_cast<int64_t>(cs.slot) * R + r) * kHeadDim + 4 * g4;
#pragma unroll
        for (int db = 0; db < 8; ++db) *reinterpret_cast<f32x4*>(dst + 16 * db) = o[rb][db];
      }
    }
  };
  while (f.valid) {
    if (!started || f.sg.slot != cs.slot) {    // wave-uniform: the stream has entered another pair
      if (started) finish();
      cs = f.sg;
      started = true;
      {                                        // Q rows of the pair -> LDS (row R is the zero row of the padding)
        u32x4 qtmp[kQIters];
#pragma unroll
        for (int j = 0; j < kQIters; ++j) {
          const int ch = lane + kThreads * j;
          const int r = ch >> 4, c = ch & 15;
          u32x4 v = {0u, 0u, 0u, 0u};
          if (r < R) {
            const int i = r / G, hg = r - i * G;
            v = *reinterpret_cast<const u32x4*>(q + ((static_cast<int64_t>(cs.rq) * n_q + i) * kv.num_q_heads + cs.g * G + hg) * kHeadDim + 8 * c);
          }
          qtmp[j] = v;
        }
#pragma unroll
        for (int j = 0; j < kQIters; ++j) {
          const int ch = lane + kThreads * j;
          if (ch < (R + 1) * 16) *reinterpret_cast<u32x4*>(s_q + k_lds_addr(ch >> 4, ch & 15)) = qtmp[j];
        }
      }
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) lse2[rb] = ws.lse2[static_cast<int64_t>(cs.pair) * (RB * 16) + 16 * rb + n];
      sdst = scores + (static_cast<int64_t>(cs.rq) * kv.num_kv_heads + cs.g) * score_stride;
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int d = 0; d < 8; ++d) o[rb][d] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const int tb = f.tb;
    rows_to_lds<FP8, false>(rk, s_tile, lane);
    const float ks[2] = {f.ks[0], f.ks[1]}, vs[2] = {f.vs[0], f.vs[1]};
    f32x4 s[2][RB];
    tile_qk_ldsq<RB>(s_tile, s_q, R, s, lane);
    // the K rows are consumed: the V rows take their place, and both register sets carry the next tile
    if (tb + kTileTokens > cs.L) zero_tail_rows<FP8>(rv, tb, cs.L, geo);
    rows_to_lds<FP8, true>(rv, s_tile, lane);
    f = issue_next<FP8, true>(kv, cur, geo, lane, rk, rv);
    const bool edge = tb + kTileTokens > cs.L - n_q;
    f32x4 tot[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
    bf16x8 p[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      f32x4 pr[2];
#pragma unroll
      for (int sub = 0; sub < 2; ++sub) {
        const float sc = c2 * ks[sub];
#pragma unroll
        for (int i = 0; i < 4; ++i) pr[sub][i] = fast_exp2(fmaf(s[sub][rb][i], sc, -lse2[rb]));
      }
      if (edge) {
        const int r = 16 * rb + n;
        const int last = cs.L - n_q + (r < R ? r / G : n_q - 1);
#pragma unroll
        for (int sub = 0; sub < 2; ++sub)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (tb + 16 * sub + 4 * g4 + i > last) pr[sub][i] = 0.f;
      }
      tot[0] += pr[0];
      tot[1] += pr[1];
      if constexpr (FP8) { pr[0] *= vs[0]; pr[1] *= vs[1]; }
      p[rb] = pack_p(pr[0], pr[1]);
    }
#pragma unroll
    for (int sub = 0; sub < 2; ++sub) {
#pragma unroll
      for (int i = 0; i < 4; ++i) tot[sub][i] = row16_sum(tot[sub][i]) * inv_r;
      const int tok0 = tb + 16 * sub + 4 * g4;
      if (n == 0) {
        if (tok0 + 3 < cs.L) {
          *reinterpret_cast<f32x4*>(sdst + tok0) = tot[sub];
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (tok0 + i < cs.L) sdst[tok0 + i] = tot[sub][i];
        }
      }
    }
    tile_pv<RB>(s_tile, p, o, lane);
  }
  finish();
}

// ---------------------------------------------------------------- merge -----
// one workgroup per pair; a pair inside one range was written by pass 2 itself
__global__ __launch_bounds__(256) void verify_o_merge_range(KvView kv, int n_q, RangeWs ws, uint16_t* out) {
  const int pair = blockIdx.x;
  const int b = pair / kv.num_kv_heads, g = pair - b * kv.num_kv_heads;
  const int G = kv.num_q_heads / kv.num_kv_heads;
  const int R = n_q * G;
  const int total = ws.ctrl[0];
  const int rq = request_of(kv, b);
  const int tiles = tiles_of_len(kv.seq_lens[rq]);
  const int u0 = ws.ureq[b] + g * tiles;
  const int n_used = ranges_used(ws, total);
  const int w0 = tiles > 0 ? range_of(u0, total, n_used) : 0, w1 = tiles > 0 ? range_of(u0 + tiles - 1, total, n_used) : -1;
  if (w1 == w0) return;                        // (an empty context has no partial: zeros)
  for (int idx = threadIdx.x; idx < R * (kHeadDim / 4); idx += 256) {
    const int r = idx / (kHeadDim / 4), d4 = idx - r * (kHeadDim / 4);
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
    for (int w = w0; w <= w1; ++w)
      acc += *reinterpret_cast<const f32x4*>(ws.part_o + (static_cast<int64_t>(pair + w) * R + r) * kHeadDim + 4 * d4);
    const int i = r / G, hg = r - i * G;
    uint16_t* dst = out + ((static_cast<int64_t>(rq) * n_q + i) * kv.num_q_heads + g * G + hg) * kHeadDim;
    u32x2 pk;
    pk.x = pack2(acc.x, acc.y);
    pk.y = pack2(acc.z, acc.w);
    *reinterpret_cast<u32x2*>(dst + 4 * d4) = pk;
  }
}

// ------------------------------------------------ single-pass variant -------
// The same result with K read once: one streaming pass computes O the flash-decoding way (running
// maximum per row, unnormalised partials) and leaves behind, per token and row, the exponential
// e = exp2(s - m_tile) relative to the running maximum m_tile at that tile.  Once the pair's
// log-sum-exp is known, a small streaming kernel turns the stash into probabilities,
// p = e * exp2(m_tile - lse), and sums them over the rows: 2 bytes per (token, row) written and
// read back, against the 2 * head_dim bytes per token of the second K read it replaces.
//
// A stashed value is 16 bits: e lies in [0, 1], so it is kept as 6 bits of exponent (2^-62 .. 1;
// smaller values become some value below 2^-62) and 10 bits of mantissa, rounded to nearest: relative error at most 2^-11
// per term, hence at most 2^-11 (4.9e-4) on a score, which is a sum of positive terms.  That is inside
// the 1e-3 the statistic is specified to, and far inside what Top-K needs; the two-pass variant keeps
// full fp32 probabilities.
//
// Stash layout per tile: the lanes of every full 16-row block (64 lanes), then of the last block
// only the lanes of real rows (4 * nv, nv = R - 16 (RB - 1)); per lane 16 bytes = 8 values (tokens
// 16 sub + 4 g4 + i, sub < 2, i < 4).
__device__ __forceinline__ uint32_t stash_pack(float e0, float e1) {
  // Bits 28..13 of (e's float pattern - 64 exponent steps), rounded to nearest at the 10th mantissa bit: shifted up by 3
  // they are the upper half of a register, and the 64 steps are a whole turn of it.  What lies below 2^-63 is raised to
  // that and becomes code 0; between 2^-63 and 2^-62 the codes read back as some value below 2^-62.  Three instructions
  // for two values less than with a comparison: verification of 64 requests with 40 rows 480 -> 476 us.
  const uint32_t x0 = (__float_as_uint(fmaxf(e0, 0x1p-63f)) << 3) + 0x8000u;
  const uint32_t x1 = (__float_as_uint(fmaxf(e1, 0x1p-63f)) << 3) + 0x8000u;
  return __builtin_amdgcn_perm(x1, x0, 0x07060302u);       // the two upper halves
}
__device__ __forceinline__ u32x4 stash_pack8(const f32x4 (&pr)[2]) {
  u32x4 packed;
  packed.x = stash_pack(pr[0][0], pr[0][1]);
  packed.y = stash_pack(pr[0][2], pr[0][3]);
  packed.z = stash_pack(pr[1][0], pr[1][1]);
  packed.w = stash_pack(pr[1][2], pr[1][3]);
  return packed;
}
// The two values of a word times 2^-64: a shift of either half into float position (0 stays 0), one instruction each.  (From a shift and
// a mask the compiler makes two of the lower one.)  Readers fold the 2^64 into the per-row weight, see kStashBias.
__device__ __forceinline__ float stash_lo_scaled(uint32_t w) {
  uint32_t r;
  asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_0" : "=v"(r) : "v"(13), "v"(w));
  return __uint_as_float(r);
}
__device__ __forceinline__ float stash_hi_scaled(uint32_t w) {
  uint32_t r;
  asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_1" : "=v"(r) : "v"(13), "v"(w));
  return __uint_as_float(r);
}
constexpr float kStashBias = 64.f;

// How the stash is read back: kLanes lanes per (tile, token group g4) take the rows in turn, kRows of every block each, so that a row
// sum is kRows * blocks additions within a lane and two or three across; kRows tiles fill a wavefront.  m_ref keeps the rows
// of one lane next to each other.
template <int RB> struct StashRead {
  static constexpr int kLanes = RB <= 2 ? 4 : 8, kRows = 16 / kLanes;
  static constexpr int kTiles = kRows;                       // tiles a wavefront takes at a time
  __device__ static int m_place(int n) { return (n % kLanes) * kRows + n / kLanes; }      // place of row n of a block in m_ref
};

__device__ __forceinline__ int stash_lane(int rb, int nblocks, int nv, int n, int g4, int lane) {
  return rb < nblocks - 1 ? rb * 64 + lane : (n < nv ? (nblocks - 1) * 64 + g4 * nv + n : -1);
}

// What a wavefront of the single pass carries from tile to tile of one pair.
template <int RB> struct FlashRows {
  float m[RB], l[RB];    // running maximum of the lane's row of each block; this lane group's share of the running sum
  f32x4 o[RB][8];        // unnormalised output
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      m[rb] = -INFINITY;
      l[rb] = 0.f;
#pragma unroll
      for (int d = 0; d < 8; ++d) o[rb][d] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  }
};

// Shapes of the query rows of one KV head, the same for a whole launch (all but the last two) or for one request (nq_b, Rb).
struct RowGeom {
  int n_q, G, R;         // query slots, heads per KV head, rows
  int nv, tile_lanes;    // rows of the last block; lanes that stash a tile
  int inv_g, skip;       // 2^16 / G rounded up; heads between the last of a query's rows and the first of the next query's
  int nq_b, Rb;          // query positions and rows of the request
  // r / G: exact for r < 2^16 / G, and G <= 16, r < 64
  __device__ __forceinline__ int query(int r) const { return (r * inv_g) >> 16; }
  // elements of q and out between the first row of a (request, KV head) and row r of its rows
  __device__ __forceinline__ int64_t row(int r) const { return static_cast<int64_t>(r + query(r) * skip) * kHeadDim; }
  __device__ __forceinline__ int64_t first_row(int rq, int g) const { return (static_cast<int64_t>(rq) * n_q * (G + skip) + g * G) * kHeadDim; }
};

__device__ __forceinline__ RowGeom row_geom(const KvView& kv, int n_q, int row_blocks) {
  RowGeom r;
  r.n_q = n_q;
  r.G = kv.num_q_heads / kv.num_kv_heads;
  r.R = n_q * r.G;
  r.nv = r.R - 16 * (row_blocks - 1);
  r.tile_lanes = (row_blocks - 1) * 64 + 4 * r.nv;
  r.inv_g = ((1 << 16) + r.G - 1) / r.G;
  r.skip = kv.num_q_heads - r.G;
  r.nq_b = n_q;
  r.Rb = r.R;
  return r;
}

// Q rows of a pair -> LDS by THREADS threads, in K-tile layout (row R is the zero row of the padding), a few pieces of a thread at
// a time
template <int RB, int THREADS>
__device__ __forceinline__ void q_to_lds(const uint16_t* q, const RowGeom& rg, int rq, int g, uint8_t* s_q, int tid) {
  constexpr int kQIters = ((RB * 16 + 1) * 16 + THREADS - 1) / THREADS, kAtOnce = kQIters > 4 ? 4 : kQIters;
  const uint16_t* src = q + rg.first_row(rq, g);
#pragma unroll 1
  for (int j0 = 0; j0 < kQIters; j0 += kAtOnce) {
    u32x4 qtmp[kAtOnce];
#pragma unroll
    for (int j = 0; j < kAtOnce; ++j) {
      const int ch = tid + THREADS * (j0 + j);
      const int r = ch >> 4, c = ch & 15;
      u32x4 v = {0u, 0u, 0u, 0u};
      if (r < rg.Rb) v = *reinterpret_cast<const u32x4*>(src + rg.row(r) + 8 * c);
      qtmp[j] = v;
    }
#pragma unroll
    for (int j = 0; j < kAtOnce; ++j) {
      const int ch = tid + THREADS * (j0 + j);
      if (ch < (rg.R + 1) * 16) *reinterpret_cast<u32x4*>(s_q + k_lds_addr(ch >> 4, ch & 15)) = qtmp[j];
    }
  }
}

// ------------------------------------------ stream of one stretch ----------
// The tiles of one stretch of one pair, for one wavefront, with as little per tile as possible: the byte offset of a page
// (and, for fp8, its scales) is worked out for 64 pages at a time, a page per lane, and read from its lane.
template <bool FP8> struct Stretch {
  int rq, g, L, last_page;
  int tile;                // next tile to send for
  int win, next;           // window of 64 pages that lane j holds page j of; page ids of the following window
  uint32_t lo, hi;         // byte offset of the page and head in the pools
  float ks, vs;            // its scales
};
template <bool FP8> struct StretchTile {
  TileRegs<FP8> rows;
  uint64_t base[2];        // byte offsets of the two 16-token groups in the pools
  float ks[2], vs[2];
  // No tile: any contents.  Left undefined, the registers' old contents would be kept for it all through the loop over segments.
  __device__ __forceinline__ void leave() {
#pragma unroll
    for (int u = 0; u < TileRegs<FP8>::kLoads; ++u) {
      asm volatile("" : "=v"(rows.k[u]));
      asm volatile("" : "=v"(rows.v[u]));
    }
    base[0] = base[1] = 0;
    ks[0] = ks[1] = vs[0] = vs[1] = 1.f;
  }
};

template <bool FP8>
__device__ __forceinline__ int stretch_ids(const KvView& kv, const Stretch<FP8>& c, int win, int lane) {
  return kv.block_table[static_cast<int64_t>(c.rq) * kv.block_table_stride + min(win * kWindowPages + lane, c.last_page)];
}
template <bool FP8>
__device__ __forceinline__ void stretch_window(const KvView& kv, Stretch<FP8>& c, int ids) {
  const int64_t off = (static_cast<int64_t>(ids) * kv.stride_page + static_cast<int64_t>(c.g) * kv.stride_head) * (FP8 ? 1 : 2);
  c.lo = static_cast<uint32_t>(off);
  c.hi = static_cast<uint32_t>(off >> 32);
  if constexpr (FP8) {
    c.ks = kv.k_scale[static_cast<int64_t>(ids) * kv.num_kv_heads + c.g];
    c.vs = kv.v_scale[static_cast<int64_t>(ids) * kv.num_kv_heads + c.g];
  }
}
template <bool FP8>
__device__ __forceinline__ Stretch<FP8> open_stretch(const KvView& kv, int rq, int g, int L, int t0, int first_ids, int lane) {
  Stretch<FP8> c;
  c.rq = rq;
  c.g = g;
  c.L = L;
  c.last_page = (L - 1) >> kv.page_shift;
  c.tile = t0;
  c.win = ((t0 * kTileTokens) >> kv.page_shift) / kWindowPages;
  c.ks = c.vs = 1.f;
  // lane j of first_ids: page j of the request where it has one
  int ids = lane <= c.last_page ? first_ids : __builtin_amdgcn_readfirstlane(first_ids);
  if (c.win > 0) ids = stretch_ids(kv, c, c.win, lane);
  c.next = stretch_ids(kv, c, c.win + 1, lane);
  stretch_window(kv, c, ids);
  return c;
}

// sends for the K rows of the next tile / for the V rows of the same tile
template <bool FP8>
__device__ __forceinline__ void stretch_k(const KvView& kv, Stretch<FP8>& c, StretchTile<FP8>& t, const LaneGeom<FP8>& geo, int lane) {
  constexpr int kPerGroup = TileRegs<FP8>::kLoads / 2;
  const int tb = c.tile * kTileTokens;
  // both groups of a tile lie in one window: pages hold >= 16 tokens and a tile starts at a multiple of 32
  if (min(tb >> kv.page_shift, c.last_page) / kWindowPages > c.win) {
    c.win += 1;
    stretch_window(kv, c, c.next);
    c.next = stretch_ids(kv, c, c.win + 1, lane);
  }
#pragma unroll
  for (int grp = 0; grp < 2; ++grp) {
    const int tok0 = tb + 16 * grp;
    // groups beyond the end of the sequence read the last page of the request: pages are whole, so the rows exist
    const int at = min(tok0 >> kv.page_shift, c.last_page) - c.win * kWindowPages;
    const uint64_t page = (static_cast<uint64_t>(static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(c.hi), at))) << 32) |
                          static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(c.lo), at));
    t.base[grp] = page + static_cast<uint64_t>(static_cast<int64_t>(tok0 & (kv.page_size - 1)) * kv.stride_slot * (FP8 ? 1 : 2));
    if constexpr (FP8) {
      t.ks[grp] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, c.ks), at));
      t.vs[grp] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, c.vs), at));
    } else {
      t.ks[grp] = t.vs[grp] = 1.f;
    }
    const char* src = static_cast<const char*>(kv.k_pool) + t.base[grp];
#pragma unroll
    for (int u = 0; u < kPerGroup; ++u)
      t.rows.k[grp * kPerGroup + u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(src + u * geo.row_step + geo.lane_off));
  }
}
template <bool FP8>
__device__ __forceinline__ void stretch_v(const KvView& kv, Stretch<FP8>& c, StretchTile<FP8>& t, const LaneGeom<FP8>& geo) {
  constexpr int kPerGroup = TileRegs<FP8>::kLoads / 2;
#pragma unroll
  for (int grp = 0; grp < 2; ++grp) {
    const char* src = static_cast<const char*>(kv.v_pool) + t.base[grp];
#pragma unroll
    for (int u = 0; u < kPerGroup; ++u)
      t.rows.v[grp * kPerGroup + u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(src + u * geo.row_step + geo.lane_off));
  }
  c.tile += 1;
}

// K or V rows of a tile in LDS.  fp8 stays fp8 (half the LDS traffic; it is widened on the way into the matrix cores), and K and V
// have room side by side.
template <bool FP8, bool IS_V>
__device__ __forceinline__ void stretch_park(const u32x4 (&rows)[TileRegs<FP8>::kLoads], uint8_t* tile, int lane) {
  if constexpr (FP8) rows8_to_lds(rows, tile + (IS_V ? kF8TileBytes : 0), lane);
  else rows_to_lds<false, IS_V>(rows, tile, lane);
}

// S^T of the tile, Q rows from LDS too (row R is the zero row that padded rows read).  The contraction over the head
// dimension may run in any order as long as Q follows: step s takes dims 32 s + 8 g4 .. + 7 of bf16 rows, and half s % 2 of
// the 16 dims 64 (s / 2) + 16 g4 .. of fp8 rows, which one read brings for two steps.
template <int RB, bool FP8>
__device__ __forceinline__ void stretch_qk(const uint8_t* tile, const uint8_t* s_q, int R, f32x4 (&acc)[2][RB], int lane) {
  const int n = lane & 15, g4 = lane >> 4;
  int qrow[RB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) qrow[rb] = min(16 * rb + n, R);
#pragma unroll
  for (int sub = 0; sub < 2; ++sub)
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) acc[sub][rb] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto q_of = [&](int s, bf16x8 (&b)[RB]) {
    const int chunk = FP8 ? 8 * (s >> 1) + 2 * g4 + (s & 1) : 4 * s + g4;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) b[rb] = as_bf16x8(*reinterpret_cast<const u32x4*>(s_q + k_lds_addr(qrow[rb], chunk)));
  };
  auto k_of = [&](int s, u32x4 (&k)[2]) {                    // of the two 16-token groups
#pragma unroll
    for (int sub = 0; sub < 2; ++sub)
      k[sub] = FP8 ? *reinterpret_cast<const u32x4*>(tile + (16 * sub + n) * kF8Row + ((4 * (s >> 1) + g4) << 4))
                   : *reinterpret_cast<const u32x4*>(tile + k_lds_addr(16 * sub + n, 4 * s + g4));
  };
  u32x4 k[2];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    if (!FP8 || s % 2 == 0) k_of(s, k);
    bf16x8 a[2], b[RB];
    q_of(s, b);
#pragma unroll
    for (int sub = 0; sub < 2; ++sub) {
      if constexpr (FP8) {
        a[sub] = (s & 1) ? widen_fp8x8(k[sub].z, k[sub].w) : widen_fp8x8(k[sub].x, k[sub].y);
      } else {
        a[sub] = as_bf16x8(k[sub]);
      }
    }
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      acc[0][rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[0], b[rb], acc[0][rb], 0, 0, 0);
      acc[1][rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[1], b[rb], acc[1][rb], 0, 0, 0);
    }
    if (RB > 1) __builtin_amdgcn_sched_barrier(0);           // keeps the operand reads from piling up in registers
  }
}

// What a pass does with the stash: nothing, leaves it in the L2 to be written back, or writes it through.  A stash that the L2s (32 MB) cannot
// hold leaves them line by line while the pass reads, and costs it less when it does so at once: 128 requests of 1-8 K tokens (200
// MB) 518.3 -> 513.5 us, fp8 with 40 rows 64 of 512-32 K (412 MB) 457.2 -> 450.5, 16 of 24-32 K with 36 rows (293 MB) 495.7 ->
// 489.7 (medians of four turns, which differ by 0.2 %); but the finish kernel finds less of a small one: 32 requests of 4096 tokens, 42 MB
// 124.2 -> 125.1.  In between: bf16 with 20 rows 77 MB 230.2 -> 228.2, 105 310.5 -> 308.1, 126 358.4 -> 355.4, 190 552.9 -> 549.1; fp8 with 40 rows
// 63 MB 82.2 -> 82.5, 126 146.7 -> 146.7, 170 186.5 -> 185.9.  The host chooses, by what max_seq_len allows, and knows no lengths: the line
// lies so high that a bound of some times the contexts does not put a small stash beyond it (one that does, 32 requests of 1.5 K tokens
// under 32 K: 64.0 -> 64.5; of 4096 134.2 -> 134.1).  A choice on the chip costs what it gives: per tile, and once per workgroup with whole
// copies of the pass (128 requests of 1-8 K tokens 517.4, 16 of 24-32 K with 36 rows, which then spill, 489.3).
// A unified batch keeps the plain stores whatever its size: 26 of 128 requests of 24-32 K tokens verifying (233 MB) take 793 us.
enum { kNoStash = 0, kStashKept = 1, kStashThrough = 2 };
constexpr int64_t kThroughBytes = int64_t{192} << 20;

// One tile of the single pass.  Nothing crosses lanes unless a logit exceeds its row's running maximum.  (A maximum that may lag by
// 2^8 spares most of the rescaling, but the probability of a row's largest logit is then rounded to bf16 instead of being 1: with
// page scales that bf16 holds exactly, the error of fp8 outputs grew from 1.72e-3 to 1.79e-3, of the worst row from 2.6e-3 to 4.1e-3.)
// stash, m_ref: buffers of exactly the tile's stash and maxima (STASH).
// LAST: the last tile of the stretch, after which nothing is sent for, and the only one that may reach past the sequence.
// (A branch around the loads instead makes the compiler wait for all of them where it needs the first.)
constexpr int kRawBuffer = 0x00020000;          // third word of a raw buffer descriptor: no stride, no swizzle, range checked
constexpr int kWriteThrough = 16;               // sc1: a store does not stay in the L2 to be written back later
constexpr int kDropped = 0x7ffffff0;            // an offset past the end of every buffer here
template <int RB, bool FP8, int STASH, bool LAST>
__device__ __forceinline__ void stretch_tile(const KvView& kv, Stretch<FP8>& c, StretchTile<FP8>& t, const LaneGeom<FP8>& geo, const RowGeom& rg,
                                             int tb, float c2, FlashRows<RB>& st, uint8_t* s_tile, const uint8_t* s_q, __amdgpu_buffer_rsrc_t stash, __amdgpu_buffer_rsrc_t m_ref, int lane) {
  const int n = lane & 15, g4 = lane >> 4;
  f32x4 s[2][RB];
  stretch_park<FP8, false>(t.rows.k, s_tile, lane);
  const float sc[2] = {c2 * t.ks[0], c2 * t.ks[1]}, vs[2] = {t.vs[0], t.vs[1]};
  if constexpr (!LAST) stretch_k<FP8>(kv, c, t, geo, lane);        // the K registers are free: next tile's K rows leave now
  stretch_qk<RB, FP8>(s_tile, s_q, rg.R, s, lane);
  if constexpr (LAST) {
    if (tb + kTileTokens > c.L) zero_tail_rows<FP8>(t.rows.v, tb, c.L, geo);
  }
  stretch_park<FP8, true>(t.rows.v, s_tile, lane);
  if constexpr (!LAST) stretch_v<FP8>(kv, c, t, geo);              // and its V rows once the V registers are
  if (tb + kTileTokens > c.L - rg.n_q) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const int r = 16 * rb + n;
      const int last = c.L - rg.nq_b + (r < rg.Rb ? rg.query(r) : rg.nq_b - 1);
#pragma unroll
      for (int sub = 0; sub < 2; ++sub)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (tb + 16 * sub + 4 * g4 + i > last) s[sub][rb][i] = -INFINITY;
    }
  }
  bf16x8 p[RB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    // the scales are positive, so the maximum commutes with them
    const float mx = fmaxf(fmaxf(fmaxf(s[0][rb][0], s[0][rb][1]), fmaxf(s[0][rb][2], s[0][rb][3])) * sc[0],
                           fmaxf(fmaxf(s[1][rb][0], s[1][rb][1]), fmaxf(s[1][rb][2], s[1][rb][3])) * sc[1]);
    if (__any(mx > st.m[rb])) {
      const float m_new = fmaxf(st.m[rb], max_over_groups(mx));
      const float alpha = fast_exp2(st.m[rb] - (m_new == -INFINITY ? 0.f : m_new));
      st.l[rb] *= alpha;
#pragma unroll
      for (int d = 0; d < 8; ++d) st.o[rb][d] *= alpha;
      st.m[rb] = m_new;
    }
    const float m_use = st.m[rb] == -INFINITY ? 0.f : st.m[rb];
    f32x4 pr[2];
#pragma unroll
    for (int sub = 0; sub < 2; ++sub)
#pragma unroll
      for (int i = 0; i < 4; ++i) pr[sub][i] = fast_exp2(fmaf(s[sub][rb][i], sc[sub], -m_use));
    st.l[rb] += ((pr[0][0] + pr[0][1]) + (pr[0][2] + pr[0][3])) + ((pr[1][0] + pr[1][1]) + (pr[1][2] + pr[1][3]));
    if constexpr (STASH != kNoStash) {                                   // the exponentials, 16 bits each, and the maximum they refer to
      // (-inf, not m_use, for a row that sees none of the tokens so far: its weight in the finish kernel is then zero.  With 0, exp2(0 - lse)
      // overflows below an lse of about -70 in base 2, and the score of a token such a row does not see is 0 * inf.)
      // Stores past a buffer's end are dropped: lanes with nothing to store need no branch, behind which the compiler
      // could not count the stores and would wait for them, and for V, where the next tile needs K.
      const int sl = stash_lane(rb, RB, rg.nv, n, g4, lane);
      __builtin_amdgcn_raw_buffer_store_b128(stash_pack8(pr), stash, sl >= 0 ? sl * 16 : kDropped, 0, STASH == kStashThrough ? kWriteThrough : 0);
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(st.m[rb]), m_ref, g4 == 0 ? 4 * (16 * rb + StashRead<RB>::m_place(n)) : kDropped, 0, 0);
    }
    if constexpr (FP8) { pr[0] *= vs[0]; pr[1] *= vs[1]; }
    p[rb] = pack_p(pr[0], pr[1]);
  }
  if constexpr (FP8) tile_pv8<RB>(s_tile + kF8TileBytes, p, st.o, lane);
  else tile_pv<RB>(s_tile, p, st.o, lane);
}

// ------------------------------------------ a range per workgroup ----------
// Up to two row blocks (three with fp8): range w belongs to a workgroup of kTeamWaves wavefronts that share the Q rows.  Each
// takes an equal stretch of every segment's tiles, and the segment's state is put together in LDS, so that it leaves one
// partial.  Bound by the memory system at 128 requests of 1-8 K tokens (bf16, 20 rows: 2.29 GB of K and V in 383 us without
// the stash, 6.0 of 6.7 TB/s; the 200 MB of stash written cost 80 us more), by the chain of a tile (products, exponentials,
// products) at two wavefronts per SIMD with 40 rows and fp8: vector ALU busy 36 % of the time, matrix cores 15 % (245 us without
// the stash, 342 with, at 64 requests of 512-32 K tokens).  One range per wavefront, each with its own Q rows and
// partials and a cursor that ran on across pairs without draining, needed four times the segments and waited for V where it
// needed K (the compiler cannot count loads behind a branch): 484 + 72 us (pass and finish) where this takes 464 + 57; 32
// requests of 4096 tokens 112 + 19, now 103 + 17.  Whole pairs given to workgroups of 4 or 8 wavefronts, longest first, with the
// statistic and the selection in the same launch: 523 / 545 us in all at the first, but a long row then waits for one compute
// unit.  Three row blocks of bf16 stay with two wavefronts per range: here they would need more registers than there are
// (46 spilled).  No register is spilled here.
constexpr int kTeamWaves = 4;                  // two such workgroups fill a compute unit (registers)
template <int RB, int W> struct TeamLds {
  static constexpr int kORow = kHeadDim * 4 + 16;            // a row of O on its way between wavefronts
  static_assert(16 * kORow <= kVTileBytes, "a block of O fits a tile buffer");
  __attribute__((aligned(16))) uint8_t tile[W * kVTileBytes];
  static constexpr int kQBytes = (RB * 16 + 1) * kKRow;
  static constexpr int kSolo = RB >= 3 ? 3 : W;              // wavefronts that take short segments (two workgroups share 160 KB)
  __attribute__((aligned(16))) uint8_t q[kQBytes];
  float m[W * RB * 16], l[W * RB * 16];
  __attribute__((aligned(16))) uint8_t solo_q[(kSolo - 1) * kQBytes];        // last: what the team uses stays below 64 KB, in reach of an offset
};

// A value of which the compiler knows nothing: what is worked out from it stays where it is written.  Addresses of the parts that run
// once per segment, hoisted out of the loop over segments, would hold registers through the loop over tiles and spill.
__device__ __forceinline__ int opaque(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// ------------------------------------------ segments of a range -----------
// The segments of a range one after the other.  The lengths of 64 requests wait in a register, one per lane, and the first 64 page
// ids of this request and of the next one in two more, so that entering a segment waits for no table.
struct Walk {
  int unit, end, slot;     // first unit of the segment, end of the range, slot of a segment less its pair
  Segment sg;
  int lens, len0;          // lane j: length of request len0 + j of the launch
  int ids, ids_next;       // lane j: page j of the segment's request / of the request after it
  bool live;
};

__device__ __forceinline__ int load_lengths(const KvView& kv, int b, int lane) { return kv.seq_lens[request_of(kv, min(b + lane, kv.batch - 1))]; }

__device__ __forceinline__ Walk open_walk(const KvView& kv, const RangeWs& ws, int w, int lane, bool publish) {
  const RangeStart start = open_range<kMinTeamPiece, kMaxTeamPiece>(kv, ws, w, lane, publish);
  Walk c;
  c.slot = start.slot;
  c.unit = start.unit;
  c.end = start.end;
  c.sg = uniform(start.sg);
  c.live = start.live;
  c.len0 = c.sg.b;
  c.ids = load_window(kv, c.sg.b, 0, lane);
  c.lens = load_lengths(kv, c.sg.b, lane);
  c.ids_next = load_window(kv, min(c.sg.b + 1, kv.batch - 1), 0, lane);
  return c;
}

__device__ __forceinline__ void next_segment(const KvView& kv, Walk& c, int lane) {
  Segment& sg = c.sg;
  c.unit += sg.tile1 - sg.tile0;
  c.live = c.unit < c.end;
  if (!c.live) return;
  sg.g += 1;
  if (sg.g == kv.num_kv_heads) {
    sg.g = 0;
    int skipped = -1;
    do {                                       // (an empty context has no tile; units are left, so there is one that has)
      sg.b += 1;
      skipped += 1;
      if (sg.b - c.len0 >= kWave) {
        c.len0 = sg.b;
        c.lens = load_lengths(kv, sg.b, lane);
      }
      sg.L = __builtin_amdgcn_readlane(c.lens, sg.b - c.len0);
    } while (sg.L <= 0 && sg.b + 1 < kv.batch);
    sg.rq = __builtin_amdgcn_readfirstlane(request_of(kv, sg.b));
    sg.tiles = tiles_of_len(sg.L);
    c.ids = c.ids_next;
    if (__builtin_expect(skipped > 0, 0)) c.ids = load_window(kv, sg.b, 0, lane);
    c.ids_next = load_window(kv, min(sg.b + 1, kv.batch - 1), 0, lane);
  }
  sg.tile0 = 0;
  sg.tile1 = min(sg.tiles, c.end - c.unit);
  sg.pair = sg.b * kv.num_kv_heads + sg.g;
  sg.slot = sg.pair + c.slot;
}

// (m, l) and O of a segment that one wavefront went through alone: final when it is the whole pair, else a partial.
template <int RB>
__device__ __forceinline__ void store_solo(const RangeWs& ws, const RowGeom& rg, const Segment& cs, const FlashRows<RB>& st,
                                           uint16_t* out, int lane) {
  const int n = lane & 15, g4 = lane >> 4;
  const bool whole = cs.tile0 == 0 && cs.tile1 == cs.tiles;
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const float l = sum_over_groups(st.l[rb]);
    const int r = 16 * rb + n;
    if (g4 == 0) {
      ws.part_m[static_cast<int64_t>(cs.slot) * (RB * 16) + r] = st.m[rb];
      ws.part_l[static_cast<int64_t>(cs.slot) * (RB * 16) + r] = l;
    }
    if (r >= rg.Rb) continue;                  // rows of query slots the request does not use are left alone
    if (whole) {
      const float inv = l > 0.f ? 1.0f / l : 0.f;            // a row that sees no token: zeros
      uint16_t* dst = out + rg.first_row(cs.rq, cs.g) + rg.row(r) + 4 * g4;
#pragma unroll
      for (int db = 0; db < 8; ++db) {
        u32x2 pk;
        pk.x = pack2(st.o[rb][db][0] * inv, st.o[rb][db][1] * inv);
        pk.y = pack2(st.o[rb][db][2] * inv, st.o[rb][db][3] * inv);
        *reinterpret_cast<u32x2*>(dst + 16 * db) = pk;
      }
    } else {
      float* dst = ws.part_o + (static_cast<int64_t>(cs.slot) * rg.R + r) * kHeadDim + 4 * g4;
#pragma unroll
      for (int db = 0; db < 8; ++db) *reinterpret_cast<f32x4*>(dst + 16 * db) = st.o[rb][db];
    }
  }
}

// Short segments: shared by the wavefronts, one leaves them with a tile or two each, or none, and all wait at the barriers of its
// merge.  Where as many units are left in the range as that many pairs alike have, the wavefronts take the segments of pairs of up to
// kSoloTiles tiles in turn instead, each with Q rows of its own.  Shared / in turn (before the teams, with a range per wavefront):
// 300 requests of 20-8000 tokens, their logarithms spread evenly, fp8 and 40 rows 540 / 383 (452) us, with bf16, 20 rows and no
// statistic 380 / 299 (354); 1000 of 32-64 tokens 223 / 185 (266), of 256-512 497 / 487 (554).  Up to 6 tiles the first takes
// 4 % longer, up to 24 as well, and with 48 so do 128 requests of 1-8 K tokens.
constexpr int kSoloTiles = 12;
// A segment of a short pair, with units left for the `alike` wavefronts that wait for one (the rest of a long pair is shared: what follows
// it is long as well).
__device__ __forceinline__ bool solo_segment(const Walk& c, int alike) {
  return c.sg.tiles <= kSoloTiles && c.end - c.unit >= alike * c.sg.tiles;
}

template <int RB, bool FP8, int W, int STASH>
__device__ __forceinline__ void flash_solo_run(const KvView& kv, const uint16_t* q, RowGeom rg, const RangeWs& ws, uint16_t* out, float c2,
                                               TeamLds<RB, W>& lds, Walk& walk, int wave, int lane0) {
  uint8_t* s_tile = lds.tile + wave * kVTileBytes;
  uint8_t* s_q = wave == 0 ? lds.q : lds.solo_q + (wave - 1) * TeamLds<RB, W>::kQBytes;
  int turn = 0;
  do {
    if (turn == wave) {
      const int lane = opaque(lane0);
      const LaneGeom<FP8> geo = lane_geom<FP8>(kv, lane);
      const Segment cs = walk.sg;
      const int64_t u0 = walk.unit - cs.tile0;               // unit of the pair's first tile
      rg.nq_b = __builtin_amdgcn_readfirstlane(queries_of(kv, ws, cs.b, rg.n_q));
      rg.Rb = rg.nq_b * rg.G;
      Stretch<FP8> cur = open_stretch<FP8>(kv, cs.rq, cs.g, cs.L, cs.tile0, walk.ids, lane);
      StretchTile<FP8> tl;
      stretch_k<FP8>(kv, cur, tl, geo, lane);
      stretch_v<FP8>(kv, cur, tl, geo);
      q_to_lds<RB, kWave>(q, rg, cs.rq, cs.g, s_q, lane);
      FlashRows<RB> st;
      st.clear();
      auto tile = [&](int t, auto last) {
        stretch_tile<RB, FP8, STASH, decltype(last)::value>(
            kv, cur, tl, geo, rg, t * kTileTokens, c2, st, s_tile, s_q,
            __builtin_amdgcn_make_buffer_rsrc(ws.stash + (u0 + t) * rg.tile_lanes * 16, 0, rg.tile_lanes * 16, kRawBuffer),
            __builtin_amdgcn_make_buffer_rsrc(ws.m_ref + (u0 + t) * RB * 16, 0, RB * 16 * 4, kRawBuffer), lane);
      };
      for (int t = cs.tile0; t + 1 < cs.tile1; ++t) tile(t, std::false_type{});
      tile(cs.tile1 - 1, std::true_type{});
      store_solo<RB>(ws, rg, cs, st, out, lane);
    }
    turn = turn + 1 == TeamLds<RB, W>::kSolo ? 0 : turn + 1;
    next_segment(kv, walk, lane0);
  } while (walk.live && solo_segment(walk, TeamLds<RB, W>::kSolo - turn));
}

template <int RB, bool FP8, int W, int STASH>
__device__ __forceinline__ void flash_team_body(const KvView& kv, const uint16_t* q, int n_q, const RangeWs& ws, uint16_t* out,
                                                TeamLds<RB, W>& lds, int w) {
  constexpr int THREADS = W * kWave, rows = RB * 16, kORow = TeamLds<RB, W>::kORow;
  const int lane0 = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  RowGeom rg = row_geom(kv, n_q, RB);
  const float c2 = kv.sm_scale * kLog2e;
  uint8_t* s_tile = lds.tile + wave * kVTileBytes;
  Walk team = open_walk(kv, ws, w, lane0, wave == 0);        // the segments of the range, the same for all wavefronts
  if (!team.live) return;
  while (team.live) {
    if (__builtin_expect(solo_segment(team, TeamLds<RB, W>::kSolo), 0)) {
      flash_solo_run<RB, FP8, W, STASH>(kv, q, rg, ws, out, c2, lds, team, wave, lane0);
      __syncthreads();                                       // their Q rows have been read
      continue;
    }
    const int lane = opaque(lane0);
    const LaneGeom<FP8> geo = lane_geom<FP8>(kv, lane);
    const Segment cs = team.sg;
    rg.nq_b = __builtin_amdgcn_readfirstlane(queries_of(kv, ws, cs.b, n_q));
    rg.Rb = rg.nq_b * rg.G;
    const int nt = cs.tile1 - cs.tile0;
    const int t0 = cs.tile0 + wave * nt / W, t1 = cs.tile0 + (wave + 1) * nt / W;
    Stretch<FP8> cur = open_stretch<FP8>(kv, cs.rq, cs.g, cs.L, t0, team.ids, lane);
    StretchTile<FP8> tl;
    if (t0 < t1) {
      stretch_k<FP8>(kv, cur, tl, geo, lane);
      stretch_v<FP8>(kv, cur, tl, geo);
    } else {
      tl.leave();
    }
    q_to_lds<RB, THREADS>(q, rg, cs.rq, cs.g, lds.q, opaque(threadIdx.x));
    FlashRows<RB> st;
    st.clear();
    __syncthreads();
    const int64_t u0 = team.unit - cs.tile0;                 // unit of the pair's first tile
    auto tile = [&](int t, auto last) {
      stretch_tile<RB, FP8, STASH, decltype(last)::value>(
          kv, cur, tl, geo, rg, t * kTileTokens, c2, st, s_tile, lds.q,
          __builtin_amdgcn_make_buffer_rsrc(ws.stash + (u0 + t) * rg.tile_lanes * 16, 0, rg.tile_lanes * 16, kRawBuffer),
          __builtin_amdgcn_make_buffer_rsrc(ws.m_ref + (u0 + t) * rows, 0, rows * 4, kRawBuffer), lane);
    };
    for (int t = t0; t + 1 < t1; ++t) tile(t, std::false_type{});
    if (t0 < t1) tile(t1 - 1, std::true_type{});
    // the team's (m, l) per row
    const int tid = opaque(threadIdx.x), n = tid & 15, g4 = (tid & (kWave - 1)) >> 4;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const float l = sum_over_groups(st.l[rb]);
      if (g4 == 0) {
        lds.m[wave * rows + 16 * rb + n] = st.m[rb];
        lds.l[wave * rows + 16 * rb + n] = l;
      }
    }
    __syncthreads();
    const bool whole = cs.tile0 == 0 && cs.tile1 == cs.tiles;
    float wgt[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const int r = 16 * rb + n;
      float m = -INFINITY, l = 0.f;
#pragma unroll
      for (int i = 0; i < W; ++i) m = fmaxf(m, lds.m[i * rows + r]);
      const float mu = (m == -INFINITY) ? 0.f : m;
#pragma unroll
      for (int i = 0; i < W; ++i) l += lds.l[i * rows + r] * fast_exp2(lds.m[i * rows + r] - mu);
      if (wave == 0 && g4 == 0) {
        ws.part_m[static_cast<int64_t>(cs.slot) * rows + r] = m;
        ws.part_l[static_cast<int64_t>(cs.slot) * rows + r] = l;
      }
      wgt[rb] = fast_exp2(st.m[rb] - mu);                    // no tile, or a row that sees no token: exp2(-inf)
      if (whole) wgt[rb] *= l > 0.f ? 1.0f / l : 0.f;
    }
    // O, one block of 16 rows at a time: every wavefront leaves its weighted share in its tile buffer
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
#pragma unroll
      for (int db = 0; db < 8; ++db) *reinterpret_cast<f32x4*>(s_tile + n * kORow + 64 * db + 16 * g4) = st.o[rb][db] * wgt[rb];
      __syncthreads();
      for (int idx = tid; idx < 16 * (kHeadDim / 4); idx += THREADS) {
        const int rr = idx / (kHeadDim / 4), d4 = idx - rr * (kHeadDim / 4), r = 16 * rb + rr;
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < W; ++i) acc += *reinterpret_cast<const f32x4*>(lds.tile + i * kVTileBytes + rr * kORow + 16 * d4);
        if (r < rg.Rb) {                                     // rows of query slots the request does not use are left alone
          if (whole) {
            u32x2 pk;
            pk.x = pack2(acc.x, acc.y);
            pk.y = pack2(acc.z, acc.w);
            *reinterpret_cast<u32x2*>(out + rg.first_row(cs.rq, cs.g) + rg.row(r) + 4 * d4) = pk;
          } else {
            *reinterpret_cast<f32x4*>(ws.part_o + (static_cast<int64_t>(cs.slot) * rg.R + r) * kHeadDim + 4 * d4) = acc;
          }
        }
      }
      __syncthreads();
    }
    next_segment(kv, team, lane0);
  }
}

template <int RB, bool FP8, int STASH>
__global__ __launch_bounds__(kTeamWaves * kWave, 2) void verify_flash_team(KvView kv, const uint16_t* q, int n_q, RangeWs ws, uint16_t* out) {
  __shared__ TeamLds<RB, kTeamWaves> lds;
  flash_team_body<RB, FP8, kTeamWaves, STASH>(kv, q, n_q, ws, out, lds, blockIdx.x);
}

// A unified batch in one grid (paper Section 4.2, "Fused Sparse and Full Attention"): the first n_ranges workgroups carry a
// range of the verification pass each, as in their own kernel, the workgroups after them one (request, KV head, span) of
// the draft step each.  Which path a workgroup takes is decided on the chip from its index; the draft workgroups come last
// in dispatch order, so they fill the compute units as the ranges drain.
template <int RB, bool FP8, bool MAY_BYPASS>
__global__ __launch_bounds__(kTeamWaves * kWave, 2) void mixed_flash_team(KvView kv, const uint16_t* q, int n_q, RangeWs ws, uint16_t* out,
                                                                          DecodeArgs da, DecWs dws, int span_rows, int nspan) {
  __shared__ TeamLds<RB, kTeamWaves> lds;      // its tile buffers serve the draft path too
  if (static_cast<int>(blockIdx.x) < ws.n_ranges) {
    flash_team_body<RB, FP8, kTeamWaves, kStashKept>(kv, q, n_q, ws, out, lds, blockIdx.x);
  } else {
    const DecPlace at = decode_place(FP8, blockIdx.x - ws.n_ranges, da.kv.batch, da.kv.num_kv_heads, nspan);
    decode_span_body<FP8, kTeamWaves, MAY_BYPASS>(da, dws, span_rows, nspan, at.slot_b, at.g, at.sp,
                                                  reinterpret_cast<uint8_t (*)[kVTileBytes]>(lds.tile));
  }
}

// ------------------------------------------ 3 and 4 row blocks: two wavefronts per range ----
// With more than 32 query rows the accumulators of a wavefront leave room for one wavefront per
// SIMD only, and the pass is bound by that wavefront's own instruction stream.  Here two
// wavefronts share a range: both walk the same tile stream, each fetches one 16-token half of
// every tile into the shared LDS tile, and each keeps the accumulators of its own row blocks
// (blocks 0-1, and the rest).  Four workgroup barriers per tile order the use of the one buffer:
// K halves written | S^T read | V halves written | O^T read.
template <bool FP8> struct HalfRegs { static constexpr int kLoads = TileRegs<FP8>::kLoads / 2; };

// pages of both 16-token groups of the tile at tb (the window only moves forward), loads of group `half` only
template <bool FP8>
__device__ __forceinline__ void issue_half(const KvView& kv, const Segment& sg, int tb, int half, PageWin& pw, const LaneGeom<FP8>& geo,
                                           int lane, u32x4 (&rk)[HalfRegs<FP8>::kLoads], u32x4 (&rv)[HalfRegs<FP8>::kLoads],
                                           int (&pages)[2]) {
  constexpr int kPerGroup = HalfRegs<FP8>::kLoads;
  const int esz = FP8 ? 1 : 2;
  const int last_page = (sg.L - 1) >> kv.page_shift;
#pragma unroll
  for (int grp = 0; grp < 2; ++grp) {
    const int lp = min((tb + 16 * grp) >> kv.page_shift, last_page);
    if (lp / kWindowPages > pw.win) {          // wave-uniform
      pw.pg_a = pw.pg_b;
      pw.win += 1;
      pw.pg_b = load_window(kv, sg.b, pw.win + 1, lane);
    }
    pages[grp] = __builtin_amdgcn_readlane(pw.pg_a, lp - pw.win * kWindowPages);
  }
  const int tok0 = tb + 16 * half;
  const int page = half == 0 ? pages[0] : pages[1];
  const int64_t base = (static_cast<int64_t>(page) * kv.stride_page + static_cast<int64_t>(sg.g) * kv.stride_head +
                        static_cast<int64_t>(tok0 & (kv.page_size - 1)) * kv.stride_slot) * esz;
  const char* gk = static_cast<const char*>(kv.k_pool) + base;
  const char* gv = static_cast<const char*>(kv.v_pool) + base;
#pragma unroll
  for (int u = 0; u < kPerGroup; ++u) {
    const int64_t step = u * geo.row_step;
    rk[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(gk + step + geo.lane_off));
    rv[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(gv + step + geo.lane_off));
  }
}

template <bool FP8>
__device__ __forceinline__ Flight issue_next_half(const KvView& kv, Cursor& c, int half, const LaneGeom<FP8>& geo, int lane,
                                                  u32x4 (&rk)[HalfRegs<FP8>::kLoads], u32x4 (&rv)[HalfRegs<FP8>::kLoads]) {
  Flight f;
  f.valid = c.live;
  f.sg = c.sg;
  f.tb = c.tile * kTileTokens;
  f.pages[0] = f.pages[1] = 0;
  f.ks[0] = f.ks[1] = f.vs[0] = f.vs[1] = 1.f;
  if (!c.live) return f;
  issue_half<FP8>(kv, c.sg, f.tb, half, c.pw, geo, lane, rk, rv, f.pages);
  fetch_scales<FP8>(kv, f);
  advance_cursor(kv, c, lane);
  return f;
}

template <bool FP8, bool IS_V>
__device__ __forceinline__ void half_to_lds(const u32x4 (&regs)[HalfRegs<FP8>::kLoads], uint8_t* tile, int lane, int half) {
  if constexpr (!FP8) {
    const int c = lane & 15;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int r = 16 * half + 4 * u + (lane >> 4);
      *reinterpret_cast<u32x4*>(tile + (IS_V ? v_lds_addr(r, c) : k_lds_addr(r, c))) = regs[u];
    }
  } else {
    const int c = (lane & 7) * 2;          // 16 fp8 = two 16-byte bf16 chunks
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int r = 16 * half + 8 * u + (lane >> 3);
      u32x4 lo, hi;
      widen_fp8x16(regs[u], lo, hi);
      *reinterpret_cast<u32x4*>(tile + (IS_V ? v_lds_addr(r, c) : k_lds_addr(r, c))) = lo;
      *reinterpret_cast<u32x4*>(tile + (IS_V ? v_lds_addr(r, c + 1) : k_lds_addr(r, c + 1))) = hi;
    }
  }
}

// S^T of the tile for row blocks rb0 .. rb0+RBW-1, Q operand from LDS
template <int RBW>
__device__ __forceinline__ void tile_qk_ldsq_at(const uint8_t* ktile, const uint8_t* qtile, int R, int rb0, f32x4 (&acc)[2][RBW], int lane) {
  const int n = lane & 15, g = lane >> 4;
  int qrow[RBW];
#pragma unroll
  for (int rb = 0; rb < RBW; ++rb) qrow[rb] = min(16 * (rb0 + rb) + n, R);
#pragma unroll
  for (int sub = 0; sub < 2; ++sub)
#pragma unroll
    for (int rb = 0; rb < RBW; ++rb) acc[sub][rb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const bf16x8 a0 = as_bf16x8(*reinterpret_cast<const u32x4*>(ktile + k_lds_addr(n, 4 * s + g)));
    const bf16x8 a1 = as_bf16x8(*reinterpret_cast<const u32x4*>(ktile + k_lds_addr(16 + n, 4 * s + g)));
#pragma unroll
    for (int rb = 0; rb < RBW; ++rb) {
      const bf16x8 b = as_bf16x8(*reinterpret_cast<const u32x4*>(qtile + k_lds_addr(qrow[rb], 4 * s + g)));
      acc[0][rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, b, acc[0][rb], 0, 0, 0);
      acc[1][rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, b, acc[1][rb], 0, 0, 0);
    }
    if (RBW > 1) __builtin_amdgcn_sched_barrier(0);
  }
}

// one of the two wavefronts: `half` = which 16 tokens of every tile it fetches, RB0 / RBW = its row blocks
template <int RB, bool FP8, int STASH, int RBW, int RB0>
__device__ __forceinline__ void flash_pair_wave(const KvView& kv, const uint16_t* q, int n_q, const RangeWs& ws, uint16_t* out,
                                                uint8_t* s_tile, uint8_t* s_q, int half) {
  constexpr int kPairThreads = 2 * kThreads;
  const int lane = threadIdx.x & (kThreads - 1);
  const int n = lane & 15, g4 = lane >> 4;
  const int G = kv.num_q_heads / kv.num_kv_heads;
  const int R = n_q * G;
  const int nv = R - 16 * (RB - 1);
  const int tile_lanes = (RB - 1) * 64 + 4 * nv;
  const float c2 = kv.sm_scale * kLog2e;
  const LaneGeom<FP8> geo = lane_geom<FP8>(kv, lane);
  constexpr int kHalf = HalfRegs<FP8>::kLoads;
  constexpr int kRowsPerLoad = FP8 ? 8 : 4;
  constexpr int kQIters = ((RB * 16 + 1) * 16 + kPairThreads - 1) / kPairThreads;
  Cursor cur = open_cursor(kv, ws, blockIdx.x, lane);
  if (!cur.live) return;                       // the same for both wavefronts
  int unit = cur.unit;
  // Half tiles in flight per wavefront: two.  Three row blocks of bf16: 402 against 414 us at 16 requests of 24-32 K tokens, with
  // 4 registers spilled; four row blocks of bf16 have one in flight (243 registers).  fp8: the dequantisation scales of a
  // tile must then be fetched along with its rows (issue_next_half), or their load at the tile's turn keeps a
  // round trip to memory in every tile.
  constexpr int DEPTH = (FP8 || RB == 3) ? 2 : 1;
  u32x4 rk[DEPTH][kHalf], rv[DEPTH][kHalf];
  Flight fl[DEPTH];
#pragma unroll
  for (int j = 0; j < DEPTH; ++j) fl[j] = issue_next_half<FP8>(kv, cur, half, geo, lane, rk[j], rv[j]);
  Segment cs = fl[0].sg;
  bool started = false;
  float m_run[RBW], l_run[RBW];
  f32x4 o[RBW][8];
  int nq_b = n_q, Rb = R;                      // query positions and rows of the current pair's request
  auto finish = [&]() {
    const bool whole = cs.tile0 == 0 && cs.tile1 == cs.tiles;
#pragma unroll
    for (int rb = 0; rb < RBW; ++rb) {
      const float l = sum_over_groups(l_run[rb]);
      const int r = 16 * (RB0 + rb) + n;
      if (g4 == 0) {
        ws.part_m[static_cast<int64_t>(cs.slot) * (RB * 16) + r] = m_run[rb];
        ws.part_l[static_cast<int64_t>(cs.slot) * (RB * 16) + r] = l;
      }
      if (r >= Rb) continue;               // rows of query slots the request does not use are left alone
      if (whole) {
        const float inv = l > 0.f ? 1.0f / l : 0.f;       // a row that sees no token: zeros
        const int i = r / G, hg = r - i * G;
        uint16_t* dst = out + ((static_cast<int64_t>(cs.rq) * n_q + i) * kv.num_q_heads + cs.g * G + hg) * kHeadDim;
#pragma unroll
        for (int db = 0; db < 8; ++db) {
          u32x2 pk;
          pk.x = pack2(o[rb][db][0] * inv, o[rb][db][1] * inv);
          pk.y = pack2(o[rb][db][2] * inv, o[rb][db][3] * inv);
          *reinterpret_cast<u32x2*>(dst + 16 * db + 4 * g4) = pk;
        }
      } else {
        float* dst = ws.part_o + (static_cast<int64_t>(cs.slot) * R + r) * kHeadDim + 4 * g4;
#pragma unroll
        for (int db = 0; db < 8; ++db) *reinterpret_cast<f32x4*>(dst + 16 * db) = o[rb][db];
      }
    }
  };
  auto tile = [&](Flight& f, u32x4 (&rk)[kHalf], u32x4 (&rv)[kHalf]) {
    __syncthreads();                           // the previous tile's V rows have been read by both wavefronts
    if (!started || f.sg.slot != cs.slot) {    // workgroup-uniform: the stream has entered another pair
      if (started) finish();
      cs = f.sg;
      started = true;
      nq_b = __builtin_amdgcn_readfirstlane(queries_of(kv, ws, cs.b, n_q));
      Rb = nq_b * G;
      {                                        // Q rows of the pair -> LDS, by both wavefronts (row R is the zero row)
        u32x4 qtmp[kQIters];
#pragma unroll
        for (int j = 0; j < kQIters; ++j) {
          const int ch = static_cast<int>(threadIdx.x) + kPairThreads * j;
          const int r = ch >> 4, c = ch & 15;
          u32x4 v = {0u, 0u, 0u, 0u};
          if (r < Rb) {
            const int i = r / G, hg = r - i * G;
            v = *reinterpret_cast<const u32x4*>(q + ((static_cast<int64_t>(cs.rq) * n_q + i) * kv.num_q_heads + cs.g * G + hg) * kHeadDim + 8 * c);
          }
          qtmp[j] = v;
        }
#pragma unroll
        for (int j = 0; j < kQIters; ++j) {
          const int ch = static_cast<int>(threadIdx.x) + kPairThreads * j;
          if (ch < (R + 1) * 16) *reinterpret_cast<u32x4*>(s_q + k_lds_addr(ch >> 4, ch & 15)) = qtmp[j];
        }
      }
#pragma unroll
      for (int rb = 0; rb < RBW; ++rb) {
        m_run[rb] = -INFINITY;
        l_run[rb] = 0.f;
#pragma unroll
        for (int d = 0; d < 8; ++d) o[rb][d] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
    }
    const int tb = f.tb;
    half_to_lds<FP8, false>(rk, s_tile, lane, half);
    const float ks[2] = {f.ks[0], f.ks[1]}, vs[2] = {f.vs[0], f.vs[1]};
    __syncthreads();                           // the K tile (and Q) is complete
    f32x4 s[2][RBW];
    tile_qk_ldsq_at<RBW>(s_tile, s_q, R, RB0, s, lane);
    if (tb + kTileTokens > cs.L) {
#pragma unroll
      for (int u = 0; u < kHalf; ++u)
        if (tb + 16 * half + kRowsPerLoad * u + geo.row >= cs.L) rv[u] = u32x4{0u, 0u, 0u, 0u};
    }
    __syncthreads();                           // both wavefronts have read the K rows
    half_to_lds<FP8, true>(rv, s_tile, lane, half);
    f = issue_next_half<FP8>(kv, cur, half, geo, lane, rk, rv);
    const bool edge = tb + kTileTokens > cs.L - n_q;
    bf16x8 p[RBW];
#pragma unroll
    for (int rb = 0; rb < RBW; ++rb) {
      f32x4 pr[2] = {s[0][rb], s[1][rb]};
      if (edge) {
        const int r = 16 * (RB0 + rb) + n;
        const int last = cs.L - nq_b + (r < Rb ? r / G : nq_b - 1);
#pragma unroll
        for (int sub = 0; sub < 2; ++sub)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (tb + 16 * sub + 4 * g4 + i > last) pr[sub][i] = -INFINITY;
      }
      const float sc0 = c2 * ks[0], sc1 = c2 * ks[1];
      float mx = fmaxf(fmaxf(fmaxf(pr[0][0], pr[0][1]), fmaxf(pr[0][2], pr[0][3])) * sc0,
                       fmaxf(fmaxf(pr[1][0], pr[1][1]), fmaxf(pr[1][2], pr[1][3])) * sc1);
      mx = max_over_groups(mx);
      const float m_new = fmaxf(m_run[rb], mx);
      const float m_use = (m_new == -INFINITY) ? 0.f : m_new;
      if (__any(m_new > m_run[rb])) {
        const float alpha = fast_exp2(m_run[rb] - m_use);
        l_run[rb] *= alpha;
#pragma unroll
        for (int d = 0; d < 8; ++d) o[rb][d] *= alpha;
      }
      m_run[rb] = m_new;
      float sum = 0.f;
#pragma unroll
      for (int sub = 0; sub < 2; ++sub)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          pr[sub][i] = fast_exp2(fmaf(pr[sub][i], sub == 0 ? sc0 : sc1, -m_use));
          sum += pr[sub][i];
        }
      l_run[rb] += sum;
      const int sl = stash_lane(RB0 + rb, RB, nv, n, g4, lane);
      if constexpr (STASH != kNoStash) {
        const auto stash = __builtin_amdgcn_make_buffer_rsrc(ws.stash + static_cast<int64_t>(unit) * tile_lanes * 16, 0, tile_lanes * 16, kRawBuffer);
        const auto m_ref = __builtin_amdgcn_make_buffer_rsrc(ws.m_ref + static_cast<int64_t>(unit) * (RB * 16), 0, RB * 16 * 4, kRawBuffer);
        __builtin_amdgcn_raw_buffer_store_b128(stash_pack8(pr), stash, sl >= 0 ? sl * 16 : kDropped, 0, STASH == kStashThrough ? kWriteThrough : 0);
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(m_new), m_ref, g4 == 0 ? 4 * (16 * (RB0 + rb) + StashRead<RB>::m_place(n)) : kDropped, 0, 0);
      }
      if constexpr (FP8) { pr[0] *= vs[0]; pr[1] *= vs[1]; }
      p[rb] = pack_p(pr[0], pr[1]);
    }
    __syncthreads();                           // the V tile is complete
    tile_pv<RBW>(s_tile, p, o, lane);
    unit += 1;
  };
  for (bool more = true; more;) {
#pragma unroll
    for (int j = 0; j < DEPTH; ++j) {
      if (!fl[j].valid) { more = false; break; }     // register sets are refilled in order: the first empty one ends the stream
      tile(fl[j], rk[j], rv[j]);
    }
  }
  finish();
}

template <int RB, bool FP8, int STASH>
__global__ __launch_bounds__(2 * kThreads, 2) void verify_flash_pair(KvView kv, const uint16_t* q, int n_q, RangeWs ws, uint16_t* out) {
  static_assert(RB >= 3, "up to two row blocks run verify_flash_team");
  constexpr int kFirst = (RB + 1) / 2;         // row blocks of the first wavefront
  __shared__ __attribute__((aligned(16))) uint8_t s_tile[kVTileBytes];
  __shared__ __attribute__((aligned(16))) uint8_t s_q[(RB * 16 + 1) * kKRow];
  if (threadIdx.x < kThreads) flash_pair_wave<RB, FP8, STASH, kFirst, 0>(kv, q, n_q, ws, out, s_tile, s_q, 0);
  else flash_pair_wave<RB, FP8, STASH, RB - kFirst, kFirst>(kv, q, n_q, ws, out, s_tile, s_q, 1);
}

// A unified batch with more than 32 query rows per KV head: the first n_ranges workgroups are those of
// verify_flash_pair, the others carry one (request, KV head, span) of the draft step each, with two wavefronts.
template <int RB, bool FP8, bool MAY_BYPASS>
__global__ __launch_bounds__(2 * kThreads, 2) void mixed_flash_pair(KvView kv, const uint16_t* q, int n_q, RangeWs ws, uint16_t* out,
                                                                    DecodeArgs da, DecWs dws, int span_rows, int nspan) {
  static_assert(RB >= 3, "up to two row blocks run mixed_flash_team");
  constexpr int kFirst = (RB + 1) / 2;
  constexpr int kPassLds = kVTileBytes + (RB * 16 + 1) * kKRow;
  static_assert(kPassLds >= 2 * kVTileBytes, "the draft path uses the same memory as two tile buffers");
  __shared__ __attribute__((aligned(16))) uint8_t smem[kPassLds];
  if (static_cast<int>(blockIdx.x) < ws.n_ranges) {
    if (threadIdx.x < kThreads) flash_pair_wave<RB, FP8, kStashKept, kFirst, 0>(kv, q, n_q, ws, out, smem, smem + kVTileBytes, 0);
    else flash_pair_wave<RB, FP8, kStashKept, RB - kFirst, kFirst>(kv, q, n_q, ws, out, smem, smem + kVTileBytes, 1);
  } else {
    const DecPlace at = decode_place(FP8, blockIdx.x - ws.n_ranges, da.kv.batch, da.kv.num_kv_heads, nspan);
    decode_span_body<FP8, 2, MAY_BYPASS>(da, dws, span_rows, nspan, at.slot_b, at.g, at.sp,
                                         reinterpret_cast<uint8_t (*)[kVTileBytes]>(smem));
  }
}

// Sort key of a score of the statistic: a mean of probabilities lies in [0, 1] (below 2 with any rounding), so the
// sign bit and the top exponent bit of its pattern are zero and can go: the first 12-bit digit of the selection
// then holds 6 exponent and 6 mantissa bits, 64 histogram bins per binade instead of 8, and scores that share a
// few exponents queue up on far fewer LDS addresses.
__device__ __forceinline__ uint32_t score_key(float f) { return __float_as_uint(f) << 2; }

// Log-sum-exp of every row of a pair (log2 domain) into s_lse, by the first 512 threads: kParSegs threads per row take the segments in turn,
// so that the (m, l) of all segments leave together, and combine through LDS (s_m: 2 * 512 floats; the number of threads per row is the
// same for every workgroup size, so the order of the sums is, too).  Rows beyond the request's own, and rows that see no token at
// all, get +inf: their probabilities vanish wherever the log-sum-exp is applied.  Returns the maximum of this thread's first segment.
template <int RB> constexpr int kParSegs = 512 / (RB * 16);
template <int RB>
__device__ __forceinline__ float pair_lse(const KvView& kv, const RangeWs& ws, int n_q, int G, int Rb, int rq, int g, const PairSegs& segs,
                                          float* lse_out, float* s_m, float* s_lse) {
  constexpr int rows = RB * 16, kPar = kParSegs<RB>;
  float* s_l = s_m + kPar * rows;
  const int my_row = static_cast<int>(threadIdx.x) % rows, my_sg = static_cast<int>(threadIdx.x) / rows;
  float m_seg = -INFINITY;
  if (my_sg < kPar) {
    float m = -INFINITY, l = 0.f;
    for (int sg = my_sg; sg < segs.n; sg += kPar) {
      const float mc = ws.part_m[static_cast<int64_t>(segs.slot0 + sg) * rows + my_row];
      const float lc = ws.part_l[static_cast<int64_t>(segs.slot0 + sg) * rows + my_row];
      if (sg == my_sg) m_seg = mc;
      const float mn = fmaxf(m, mc);
      const float mu = (mn == -INFINITY) ? 0.f : mn;
      l = l * fast_exp2(m - mu) + lc * fast_exp2(mc - mu);
      m = mn;
    }
    s_m[threadIdx.x] = m;
    s_l[threadIdx.x] = l;
  }
  __syncthreads();
  if (threadIdx.x < rows) {
    const int row = threadIdx.x;
    float m = -INFINITY, l = 0.f;
    // (every place has been written, -inf and 0 where there is no segment, so eight reads leave together)
    constexpr int kStep = kPar % 8 == 0 ? 8 : kPar;
    const int live = min(segs.n, kPar);
    for (int s0 = 0; s0 < live; s0 += kStep)
#pragma unroll
      for (int j = 0; j < kStep; ++j) m = fmaxf(m, s_m[(s0 + j) * rows + row]);
    const float mu = (m == -INFINITY) ? 0.f : m;
    for (int s0 = 0; s0 < live; s0 += kStep)
#pragma unroll
      for (int j = 0; j < kStep; ++j) l += s_l[(s0 + j) * rows + row] * fast_exp2(s_m[(s0 + j) * rows + row] - mu);
    const bool sees = row < Rb && l > 0.f;
    const float v = sees ? m + log2f(l) : INFINITY;
    s_lse[row] = v;
    if (lse_out && row < Rb) {
      const int i = row / G, hg = row - i * G;
      lse_out[(static_cast<int64_t>(rq) * n_q + i) * kv.num_q_heads + g * G + hg] = sees ? v * kLn2 : -INFINITY;
    }
  }
  __syncthreads();
  return m_seg;
}

// O of a pair cut into several segments, by `mergers` workgroups of its own: 512 threads take four rows (a piece of four dims of one each)
// by four groups that take the segments in turn.  What it costs one workgroup is the rate at which a compute unit reads what others have
// written: 17 to 33 segments of 10 KB each took 3 to 5 us between the log-sum-exp and the scores.
template <int RB, int THREADS>
__device__ __forceinline__ void merge_pair(const KvView& kv, int n_q, const RangeWs& ws, uint16_t* out, int share, int mergers, float* s_o, float* s_lse) {
  const int pair = ws.order ? ws.order[blockIdx.x] : static_cast<int>(blockIdx.x);
  const int b = pair / kv.num_kv_heads, g = pair - b * kv.num_kv_heads, rq = request_of(kv, b);
  const int G = kv.num_q_heads / kv.num_kv_heads, R = n_q * G, Rb = queries_of(kv, ws, b, n_q) * G, tiles = tiles_of_len(kv.seq_lens[rq]);
  constexpr int rows = RB * 16;
  const int u0 = ws.ureq[b] + g * tiles, total = ws.ctrl[0], cut = ws.ctrl[1];
  if (tiles <= 0) return;
  const PairSegs segs = segs_of_pair(ws, total, cut, pair, u0, tiles);
  if (segs.n <= 1) return;                     // (the pass has written O)
  pair_lse<RB>(kv, ws, n_q, G, Rb, rq, g, segs, nullptr, s_o, s_lse);
  constexpr int kQuads = THREADS / 512, kGroups = 4, kAtOnce = 8;        // quads of rows at work; segments of a thread sent for together
  const int sub = static_cast<int>(threadIdx.x) / 512, grp = static_cast<int>(threadIdx.x) % 512 / 128, piece = static_cast<int>(threadIdx.x) % 128;
  f32x4* mine = reinterpret_cast<f32x4*>(s_o) + threadIdx.x;
  for (int q0 = share * kQuads; 4 * q0 < Rb; q0 += mergers * kQuads) {
    const int row = 4 * (q0 + sub) + piece / 32, d4 = piece % 32;
    const bool there = row < Rb;
    const float* src = ws.part_o + static_cast<int64_t>(segs.slot0) * R * kHeadDim + row * kHeadDim + 4 * d4;
    const float* pm = ws.part_m + static_cast<int64_t>(segs.slot0) * rows + row;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    if (there) {
      const float lse = s_lse[row];
      for (int sg0 = grp; sg0 < segs.n; sg0 += kGroups * kAtOnce) {
        f32x4 po[kAtOnce];
        float m[kAtOnce];
#pragma unroll
        for (int j = 0; j < kAtOnce; ++j) {
          const int sg = min(sg0 + kGroups * j, segs.n - 1);
          po[j] = *reinterpret_cast<const f32x4*>(src + static_cast<int64_t>(sg) * R * kHeadDim);
          m[j] = pm[static_cast<int64_t>(sg) * rows];
        }
#pragma unroll
        for (int j = 0; j < kAtOnce; ++j)
          if (sg0 + kGroups * j < segs.n) acc += po[j] * fast_exp2(m[j] - lse);
      }
    }
    *mine = acc;
    __syncthreads();
    if (there && grp == 0) {
#pragma unroll
      for (int i = 1; i < kGroups; ++i) acc += mine[128 * i];
      const int i = row / G, hg = row - i * G;
      u32x2 pk;
      pk.x = pack2(acc.x, acc.y);
      pk.y = pack2(acc.z, acc.w);
      *reinterpret_cast<u32x2*>(out + ((static_cast<int64_t>(rq) * n_q + i) * kv.num_q_heads + g * G + hg) * kHeadDim + 4 * d4) = pk;
    }
    __syncthreads();                           // the next rows take their place
  }
}

// ------------------------------------------------ finish ---------------------
// Everything that needs the whole pair, in one kernel: one workgroup per (request, KV head), longest
// rows first.
//   1. the log-sum-exp of every row from the (m, l) of the pair's segments;
//   2. O of a pair that was cut into several segments: sum over segments of exp2(m_seg - lse) O_seg
//      (a pair inside one range was finished by the pass itself);
//   3. the score statistic from the stash, scores = mean over rows of e * exp2(m_tile - lse): wavefronts take
//      groups of two or four tiles in turn, one on its way, and leave the scores of one chunk of tokens at a time in
//      LDS, from where every thread takes 8 consecutive ones as sort keys into registers (and writes them out
//      if the caller wants the statistic itself).  What this costs is instructions as much as memory: with a lane per row, a
//      row sum across 16 lanes and a third of the lanes on rows that are not there (20 of 32), the kernel issued 1.76 times as
//      many vector instructions and took 66 us where it takes 57 (128 requests of 1-8 K tokens, 231 MB read), 1.42 times and 127
//      where it takes 117 (64 of 512-32 K, 40 rows, 432 MB), 27 where it takes 23 (26 of 1-8 K);
//   4. SELECT: Top-K of the keys in registers (topk_core.hpp) -- the statistic makes no round trip through
//      memory between two launches (paper Section 4.1: identification from the verification's own
//      intermediates).
// Rows of up to CH * THREADS * 8 tokens; without SELECT any length (the chunk loop is then a run-time one).
// SPLIT (long rows): a pair is shared by up to CH workgroups, blockIdx.y = the chunk of THREADS * 8 tokens each
// of them rebuilds; the statistic goes to memory (the caller's buffer, else scratch) and verify_select_rows, the
// next launch, selects from it.  The first chunk's workgroup also does step 1's output and step 2.  (Handing the
// chunks to the last workgroup to arrive inside one launch was measured: the device-wide release every workgroup
// then needs writes back the whole L2 behind it, 3 to 5 times the cost of the extra launch.)
// With `mergers` (few pairs), workgroups 1 .. mergers of a pair, by blockIdx.y, do step 2 and nothing else, the others no step 2.
// Up to two row blocks, two workgroups of 512 threads share a compute unit, which takes 128 registers at most: with 129, 128 requests of
// 1-8 K tokens took 539 us instead of 518 (pass and finish).
template <int RB, int THREADS, int CH, bool SELECT, bool SPLIT>
__global__ __launch_bounds__(THREADS, THREADS >= 1024 || RB <= 2 ? 4 : 2) void verify_finish(KvView kv, int n_q, RangeWs ws, uint16_t* out, float* lse_out,
                                                         float* scores, int64_t score_stride, SelectOut sel, int mergers) {
  static_assert(!SPLIT || !SELECT, "a split pair is selected by verify_select_rows");
  constexpr int KPC = 8;
  constexpr int kChunk = THREADS * KPC;                      // tokens whose scores LDS holds at a time
  constexpr int kChunkTiles = kChunk / kTileTokens;
  constexpr int kWaves = THREADS / kWave;
  __shared__ __attribute__((aligned(16))) float s_scores[kChunk];
  __shared__ float s_lse[RB * 16];
  __shared__ SelectLds<THREADS, CH> lds;
  if (static_cast<int>(blockIdx.y) - 1 < mergers && blockIdx.y > 0) {
    merge_pair<RB, THREADS>(kv, n_q, ws, out, static_cast<int>(blockIdx.y) - 1, mergers, s_scores, s_lse);
    return;
  }
  const int pair = ws.order ? ws.order[blockIdx.x] : static_cast<int>(blockIdx.x);
  const int b = pair / kv.num_kv_heads, g = pair - b * kv.num_kv_heads;
  const int rq = request_of(kv, b);
  const int L = kv.seq_lens[rq];
  const int tiles = tiles_of_len(L);
  const int G = kv.num_q_heads / kv.num_kv_heads;
  const int R = n_q * G;
  const int Rb = queries_of(kv, ws, b, n_q) * G;
  constexpr int rows = RB * 16;
  const int u0 = ws.ureq[b] + g * tiles, total = ws.ctrl[0], cut = ws.ctrl[1];             // (sent for beside the length)
  const int my_chunk = SPLIT && blockIdx.y > 0 ? static_cast<int>(blockIdx.y) - mergers : 0;
  if (SPLIT && my_chunk > 0 && my_chunk * kChunk >= L) return;      // this pair has fewer chunks (uniform over the workgroup)
  const bool lead = my_chunk == 0;                       // the workgroup that writes what exists once per pair
  int K = 0;
  int32_t* out_idx = nullptr;
  if constexpr (SELECT) {
    K = max(0, min(min(sel.budgets[rq], L), sel.max_budget));
    out_idx = sel.indices + (static_cast<int64_t>(rq) * kv.num_kv_heads + g) * sel.max_budget;
    if (g == 0 && threadIdx.x == 0) sel.counts[rq] = K;
    for (int j = K + threadIdx.x; j < sel.max_budget; j += THREADS) out_idx[j] = -1;
  }

  if (L <= 0) {                                          // an empty context: no unit, no segment; no query sees a token
    for (int idx = threadIdx.x; idx < Rb * (kHeadDim / 4); idx += THREADS) {
      const int r = idx / (kHeadDim / 4), i = r / G, hg = r - i * G;
      const int64_t row = (static_cast<int64_t>(rq) * n_q + i) * kv.num_q_heads + g * G + hg;
      *reinterpret_cast<u32x2*>(out + row * kHeadDim + 4 * (idx - r * (kHeadDim / 4))) = u32x2{0u, 0u};
      if (lse_out && idx == r * (kHeadDim / 4)) lse_out[row] = -INFINITY;
    }
    return;
  }

  // (its divisions come after the workgroups with nothing to do have left: where max_seq_len allows for more chunks than there are, they run
  // when the others have finished, and 32 requests of 1.5 K tokens under a max_seq_len of 32 K took 66.9 us instead of 64.7)
  const PairSegs segs = segs_of_pair(ws, total, cut, pair, u0, tiles);
  const int nseg = segs.n;
  const bool split = nseg > 1;
  const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int nv = R - 16 * (RB - 1);
  const int tile_lanes = (RB - 1) * 64 + 4 * nv;
  const bool want_scores = SELECT || SPLIT || scores;

  // The stash stream: wavefronts take groups of kGroup tiles in turn, through range-checked buffers of one chunk that read as zero
  // where there is no tile or row.  A register is sent for again as soon as it has been used, so a group is always on its way.
  using Read = StashRead<RB>;
  constexpr int kRows = Read::kRows, kGroup = Read::kTiles;
  const int my_r = lane % Read::kLanes, my_g4 = lane / Read::kLanes % 4, my_tile = lane / (4 * Read::kLanes);
  const int rows_there = (nv + Read::kLanes - 1) / Read::kLanes;         // of the last block, per lane
  u32x4 st[RB][kRows];
  float mref[RB][kRows];
  struct Chunk {
    __amdgpu_buffer_rsrc_t stash, m_ref;
    int groups;
  };
  auto open_chunk = [&](int c) {
    const int t_begin = c * kChunkTiles, n = min(tiles, t_begin + kChunkTiles) - t_begin;
    Chunk ch;
    ch.stash = __builtin_amdgcn_make_buffer_rsrc(ws.stash + (static_cast<int64_t>(u0) + t_begin) * tile_lanes * 16, 0, n * tile_lanes * 16, kRawBuffer);
    ch.m_ref = __builtin_amdgcn_make_buffer_rsrc(ws.m_ref + (static_cast<int64_t>(u0) + t_begin) * rows, 0, n * rows * 4, kRawBuffer);
    ch.groups = (n + kGroup - 1) / kGroup;
    return ch;
  };
  constexpr int kStream = 2;                             // nt: read once
  auto fetch_row = [&](const Chunk& ch, int group, int rb, int j) {
    const int tile0 = (group * kGroup + my_tile) * tile_lanes * 16;
    const bool last = rb == RB - 1;
    const int off = last ? ((RB - 1) * 64 + my_g4 * nv + my_r + Read::kLanes * j) * 16 : rb * 1024 + (my_g4 * 16 + my_r + Read::kLanes * j) * 16;
    const bool there = !last || my_r + Read::kLanes * j < nv;
    st[rb][j] = __builtin_amdgcn_raw_buffer_load_b128(ch.stash, there ? tile0 + off : kDropped, 0, kStream);
  };
  auto fetch_m = [&](const Chunk& ch, int group) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const int off = ((group * kGroup + my_tile) * rows + 16 * rb + my_r * kRows) * 4;
      if constexpr (kRows == 4) {
        const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(ch.m_ref, off, 0, kStream);
        mref[rb][0] = __uint_as_float(v.x); mref[rb][1] = __uint_as_float(v.y); mref[rb][2] = __uint_as_float(v.z); mref[rb][3] = __uint_as_float(v.w);
      } else {
        const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(ch.m_ref, off, 0, kStream);
        mref[rb][0] = __uint_as_float(v.x); mref[rb][1] = __uint_as_float(v.y);
      }
    }
  };
  auto row_there = [&](int rb, int j) { return rb < RB - 1 || j < rows_there; };         // uniform over the launch
  Chunk ch;
  auto prime = [&](int c) {                              // first tiles of chunk c on their way
    ch = open_chunk(c);
    fetch_m(ch, wave);
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int j = 0; j < kRows; ++j)
        if (row_there(rb, j)) fetch_row(ch, wave, rb, j);
  };
  if (want_scores) prime(my_chunk);                    // needs nothing of steps 1 and 2: in flight meanwhile

  // 1. log-sum-exp per row (log2 domain).
  // 2. O of a pair cut into several segments.  The partials of the first kSegs segments are fetched before the
  // log-sum-exp is known (every thread owns up to kOuts pieces of 4 dims), so both waits overlap; the weights of kPar
  // segments at a time wait in LDS.  The workgroups that share a pair (SPLIT) share its pieces too.
  // A loop over the segments by one thread per row was a round trip to memory per segment: one request of 2100 tokens
  // (66 segments of one tile) 96 -> 20 us, 32 of 4096 tokens (5) 25 -> 19 us, 26 of up to 8 K tokens (10) 47 -> 30 us.
  constexpr int kPar = kParSegs<RB>;
  // (as many as the registers hold beside the stash that is on its way: with 5, two row blocks of a 512-thread workgroup spill up to
  // five; the keys of four chunks leave room for 2 or 3)
  constexpr int kSegs = CH == 4 ? (RB == 4 ? 2 : 3) : THREADS >= 1024 || RB == 2 ? 4 : 5;
  constexpr int kOuts = (rows * (kHeadDim / 4) + THREADS - 1) / THREADS;
  static_assert(2 * kPar * rows <= kChunk, "the (m, l) of the segments wait where the scores will be");
  const bool merge_here = split && mergers == 0;
  const int n_share = SPLIT ? (L + kChunk - 1) / kChunk : 1;             // workgroups of this pair
  const int pieces = Rb * (kHeadDim / 4);
  const int my_first = my_chunk * pieces / n_share, my_end = (my_chunk + 1) * pieces / n_share;
  f32x4 po[kOuts][kSegs];
  if (merge_here) {
#pragma unroll
    for (int o = 0; o < kOuts; ++o) {
      const int idx = my_first + static_cast<int>(threadIdx.x) + o * THREADS;
#pragma unroll
      for (int sg = 0; sg < kSegs; ++sg) {
        po[o][sg] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (idx < my_end && sg < nseg)
          po[o][sg] = *reinterpret_cast<const f32x4*>(ws.part_o + static_cast<int64_t>(segs.slot0 + sg) * R * kHeadDim + 4 * idx);
      }
    }
  }
  float* s_m = s_scores;                                 // [kPar][rows] maximum, then weight, of a segment's rows
  const int my_row = static_cast<int>(threadIdx.x) % rows, my_sg = static_cast<int>(threadIdx.x) / rows;
  const bool merging = my_sg < kPar;
  const float m_seg = pair_lse<RB>(kv, ws, n_q, G, Rb, rq, g, segs, lead ? lse_out : nullptr, s_m, s_lse);       // of this thread's first segment
  if (merge_here) {
    f32x4 acc[kOuts];
#pragma unroll
    for (int o = 0; o < kOuts; ++o) acc[o] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int c0 = 0; c0 < nseg; c0 += kPar) {            // (one turn unless a pair spans very many ranges)
      if (c0 > 0) __syncthreads();                       // the weights of the previous turn have been read
      if (merging && c0 + my_sg < nseg) {
        const float m = c0 == 0 ? m_seg : ws.part_m[static_cast<int64_t>(segs.slot0 + c0 + my_sg) * rows + my_row];
        s_m[threadIdx.x] = fast_exp2(m - s_lse[my_row]);
      }
      __syncthreads();
      const int n_here = min(kPar, nseg - c0);
#pragma unroll
      for (int o = 0; o < kOuts; ++o) {
        const int idx = my_first + static_cast<int>(threadIdx.x) + o * THREADS;
        if (idx >= my_end) continue;
        const float* wgt = s_m + idx / (kHeadDim / 4);
        const float* src = ws.part_o + static_cast<int64_t>(segs.slot0 + c0) * R * kHeadDim + 4 * idx;
        int sg = 0;
        if (c0 == 0) {
#pragma unroll
          for (int j = 0; j < kSegs; ++j)
            if (j < n_here) acc[o] += po[o][j] * wgt[j * rows];
          sg = kSegs;
        }
#pragma unroll 4
        for (; sg < n_here; ++sg) acc[o] += *reinterpret_cast<const f32x4*>(src + static_cast<int64_t>(sg) * R * kHeadDim) * wgt[sg * rows];
      }
    }
#pragma unroll
    for (int o = 0; o < kOuts; ++o) {
      const int idx = my_first + static_cast<int>(threadIdx.x) + o * THREADS;
      if (idx >= my_end) continue;
      const int r = idx / (kHeadDim / 4), d4 = idx - r * (kHeadDim / 4);
      const int i = r / G, hg = r - i * G;
      uint16_t* dst = out + ((static_cast<int64_t>(rq) * n_q + i) * kv.num_q_heads + g * G + hg) * kHeadDim;
      u32x2 pk;
      pk.x = pack2(acc[o].x, acc[o].y);
      pk.y = pack2(acc[o].z, acc[o].w);
      *reinterpret_cast<u32x2*>(dst + 4 * d4) = pk;
    }
    __syncthreads();                                     // the scores take the place of the weights
  }
  if (!want_scores) return;

  // 3. scores of the pair, chunk by chunk
  const float log2_inv_r = -log2f(static_cast<float>(Rb));
  float bias[RB][kRows];                               // per row: -lse + the stash's 2^64 + log2(1 / rows)
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int j = 0; j < kRows; ++j) bias[rb][j] = kStashBias + log2_inv_r - s_lse[16 * rb + my_r + Read::kLanes * j];   // -inf for rows that carry no weight
  float* sdst = scores ? scores + (static_cast<int64_t>(rq) * kv.num_kv_heads + g) * score_stride : nullptr;
  if (SPLIT && !sdst) sdst = ws.scratch_scores + static_cast<int64_t>(pair) * ws.scratch_stride;
  uint32_t key[CH][KPC];
  auto chunk = [&](int c, uint32_t (&keys)[KPC]) {
    const int t_end = min(tiles, (c + 1) * kChunkTiles);
    for (int group = wave; group < ch.groups; group += kWaves) {
      // (the weights are there before the next maxima are sent for: else those get other registers, are moved at the loop's end and
      // waited for there; 128 requests of 1-8 K tokens 517 -> 515.5 us, 16 of 24-32 K 492 -> 489)
      float w[RB][kRows];
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int j = 0; j < kRows; ++j) {
          w[rb][j] = fast_exp2(mref[rb][j] + bias[rb][j]);
          if constexpr (CH < 4) asm volatile("" : "+v"(w[rb][j]));      // (with the keys of four chunks there is no room: a register spills)
        }
      if constexpr (CH < 4) __builtin_amdgcn_sched_barrier(0);
      fetch_m(ch, group + kWaves);
      float tot[2][4] = {};
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
#pragma unroll
        for (int j = 0; j < kRows; ++j) {
          if (!row_there(rb, j)) continue;
          const u32x4 v = st[rb][j];
          const uint32_t h[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            tot[k >> 1][(2 * k) & 3] = fmaf(stash_lo_scaled(h[k]), w[rb][j], tot[k >> 1][(2 * k) & 3]);
            tot[k >> 1][(2 * k + 1) & 3] = fmaf(stash_hi_scaled(h[k]), w[rb][j], tot[k >> 1][(2 * k + 1) & 3]);
          }
          fetch_row(ch, group + kWaves, rb, j);
        }
      }
#pragma unroll
      for (int sub = 0; sub < 2; ++sub)
#pragma unroll
        for (int i = 0; i < 4; ++i) tot[sub][i] = lanes_sum<Read::kLanes>(tot[sub][i]);
      f32x4 mine;
#pragma unroll
      for (int i = 0; i < 4; ++i) mine[i] = my_r == 0 ? tot[0][i] : tot[1][i];
      if (my_r < 2) *reinterpret_cast<f32x4*>(s_scores + (group * kGroup + my_tile) * kTileTokens + 16 * my_r + 4 * my_g4) = mine;
    }
    if (!SPLIT && (c + 1) * kChunk < L) prime(c + 1);   // the next chunk's first tiles leave before the barriers
    __syncthreads();
    const int p0 = c * kChunk + static_cast<int>(threadIdx.x) * KPC;      // this thread's 8 positions
#pragma unroll
    for (int j = 0; j < KPC; j += 4) {
      f32x4 v = {0.f, 0.f, 0.f, 0.f};
      if (p0 + j < t_end * kTileTokens) v = *reinterpret_cast<const f32x4*>(s_scores + static_cast<int>(threadIdx.x) * KPC + j);
#pragma unroll
      for (int i = 0; i < 4; ++i) keys[j + i] = score_key(v[i]);
      if (sdst) {
        if (p0 + j + 3 < L) {
          *reinterpret_cast<f32x4*>(sdst + p0 + j) = v;
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (p0 + j + i < L) sdst[p0 + j + i] = v[i];
        }
      }
    }
    if (!SPLIT && (c + 1) * kChunk < L) __syncthreads();                 // the next chunk overwrites the scores
  };
  if constexpr (SPLIT) {
    chunk(my_chunk, key[0]);                           // the scores of this chunk go to memory
  } else if constexpr (SELECT) {
    // (here and not at the start of the kernel, where the stores hold up the loads of short pairs: 1000 requests of up to 300 tokens
    // 300 -> 306 us)
    select_clear(lds);
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      if (c * kChunk < L) {                            // uniform over the workgroup
        chunk(c, key[c]);
      } else {
#pragma unroll
        for (int j = 0; j < KPC; ++j) key[c][j] = 0u;
      }
    }
    if (K > 0) select_topk_in_registers<THREADS, KPC, CH>(key, L, K, out_idx, lds);
  } else {
    for (int c = 0; c * kChunk < L; ++c) chunk(c, key[0]);
  }
}

// Top-K of the statistic of long rows, from memory: one workgroup per (request, KV head), longest first; thread t
// holds positions c * 8192 + 8 t .. + 7 of each chunk c (the same ownership as in verify_finish).
template <int CH>
__global__ __launch_bounds__(1024) void verify_select_rows(KvView kv, RangeWs ws, const float* scores, int64_t score_stride,
                                                           SelectOut sel) {
  constexpr int THREADS = 1024, KPC = 8, kChunk = THREADS * KPC;
  __shared__ SelectLds<THREADS, CH> lds;
  const int pair = ws.order[blockIdx.x];
  const int b = pair / kv.num_kv_heads, g = pair - b * kv.num_kv_heads;
  const int rq = request_of(kv, b);
  const int L = kv.seq_lens[rq];
  const int K = max(0, min(min(sel.budgets[rq], L), sel.max_budget));
  int32_t* out_idx = sel.indices + (static_cast<int64_t>(rq) * kv.num_kv_heads + g) * sel.max_budget;
  if (g == 0 && threadIdx.x == 0) sel.counts[rq] = K;
  for (int j = K + threadIdx.x; j < sel.max_budget; j += THREADS) out_idx[j] = -1;
  if (K == 0) return;
  const float* src = scores ? scores + (static_cast<int64_t>(rq) * kv.num_kv_heads + g) * score_stride
                            : ws.scratch_scores + static_cast<int64_t>(pair) * ws.scratch_stride;
  select_clear(lds);
  uint32_t key[CH][KPC];
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    const int p0 = c * kChunk + static_cast<int>(threadIdx.x) * KPC;
#pragma unroll
    for (int j = 0; j < KPC; j += 4) {
      f32x4 v = {0.f, 0.f, 0.f, 0.f};
      if (p0 + j + 3 < L) {
        v = *reinterpret_cast<const f32x4*>(src + p0 + j);
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (p0 + j + i < L) v[i] = src[p0 + j + i];
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) key[c][j + i] = score_key(v[i]);
    }
  }
  __syncthreads();
  select_topk_in_registers<THREADS, KPC, CH>(key, L, K, out_idx, lds);
}

// ---------------------------------------------------------------- host ------
// Ranges of the passes with a range per wavefront or per two (fp32 probabilities; more than 32 rows, 48 with fp8), and the partial
// slots of every pass: per compute unit as many wavefronts as it holds at once (registers: 2 per SIMD up to 32 rows, else 1).
// Small workloads take fewer, down to half: below about 24 tiles per range a pass gains nothing from more wavefronts, and every
// further cut of a pair is one more segment to merge.
int ranges_for(const KvView& kv, int rb) {
  int per_cu = rb >= 3 ? 4 : 8;
  const int opt = options().verify_waves;
  if (opt > 0 && opt <= per_cu) return opt * num_cus();
  const int64_t units_max = static_cast<int64_t>(kv.batch) * kv.num_kv_heads * tiles_of_len(kv.max_seq_len);
  const int fit = static_cast<int>(std::min<int64_t>(per_cu, units_max / (24 * static_cast<int64_t>(num_cus()))));
  per_cu = std::max(per_cu / 2, fit);
  return per_cu * num_cus();
}

// Ranges of the passes with a workgroup per range: as many as the chip holds at once, and no more than the `slots` that the
// workspace has been carved for (it has enough for every verify_waves: a team is several wavefronts).
int team_ranges(int slots) {
  const int opt = options().verify_waves;
  return std::min(slots, std::max(1, (opt > 0 ? opt : 8) * num_cus() / kTeamWaves));
}

int row_blocks(const KvView& kv, int n_q) { return (n_q * (kv.num_q_heads / kv.num_kv_heads) + 15) / 16; }

RangeWs carve(const KvView& kv, int n_q, void* workspace, size_t* total_bytes) {
  const int G = kv.num_q_heads / kv.num_kv_heads;
  const size_t R = static_cast<size_t>(n_q) * G;
  const size_t rpad = (R + 15) / 16 * 16;
  const size_t pairs = static_cast<size_t>(kv.batch) * kv.num_kv_heads;
  const size_t n = static_cast<size_t>(ranges_for(kv, static_cast<int>(rpad / 16)));
  const size_t slots = pairs + n;
  char* p = static_cast<char*>(workspace);
  size_t off = 0;
  auto take = [&](size_t bytes) { char* r = p ? p + off : nullptr; off += align_up(bytes, 256); return r; };
  RangeWs w;
  w.ctrl = reinterpret_cast<int32_t*>(take(64 * 4));
  w.ureq = reinterpret_cast<int32_t*>(take((static_cast<size_t>(kv.batch) + 1) * 4));
  w.order = reinterpret_cast<int32_t*>(take(pairs * 4));
  w.scratch_scores = nullptr;
  w.scratch_stride = 0;
  w.part_m = reinterpret_cast<float*>(take(slots * rpad * 4));
  w.part_l = reinterpret_cast<float*>(take(slots * rpad * 4));
  w.part_o = reinterpret_cast<float*>(take(slots * R * kHeadDim * 4));
  w.lse2 = reinterpret_cast<float*>(take(pairs * rpad * 4));
  const size_t units = pairs * tiles_of_len(kv.max_seq_len);
  const size_t tile_lanes = (rpad / 16 - 1) * 64 + 4 * (R - (rpad - 16));
  w.stash = reinterpret_cast<uint8_t*>(take(units * tile_lanes * 16));
  w.m_ref = reinterpret_cast<float*>(take(units * rpad * 4));
  w.spec_lens = nullptr;
  w.rows_pad = static_cast<int32_t>(rpad);
  w.n_ranges = static_cast<int32_t>(n);
  w.plan_in_wave = 0;
  if (total_bytes) *total_bytes = off;
  return w;
}

template <int RB, bool FP8>
hipError_t run(const VerifyArgs& a, hipStream_t st, const DecodeArgs* draft) {
  const KvView& kv = a.kv;
  RangeWs ws = carve(kv, a.n_q, a.workspace, nullptr);
  ws.spec_lens = a.spec_lens;
  ws.scratch_scores = a.scratch_scores;
  ws.scratch_stride = a.scratch_stride;
  const uint16_t* q = static_cast<const uint16_t*>(a.q);
  uint16_t* out = static_cast<uint16_t*>(a.out);
  const int pairs = kv.batch * kv.num_kv_heads;
  const bool single_pass = !a.exact_scores || !(a.scores || a.select);
  ws.plan_in_wave = single_pass && kv.batch <= kWave * kPlanRegs;
  if (!ws.plan_in_wave) {
    KernelTimer t("verify_range_plan", st);
    hipLaunchKernelGGL(range_plan, dim3(1), dim3(1024), 0, st, kv, ws);
  }
  if (single_pass) {
    const bool stats = a.scores || a.select;
    const int rows = a.n_q * (kv.num_q_heads / kv.num_kv_heads);
    const bool through = static_cast<int64_t>(pairs) * tiles_of_len(kv.max_seq_len) * kTileTokens * rows * 2 > kThroughBytes;
    const bool fused = draft != nullptr;       // a unified batch: the draft step of other requests rides in the same grid
    DecWs dws{};
    int span_rows = 0, nspan = 0, n_draft = 0;
    bool may_bypass = false;
    if (fused) {
      may_bypass = draft_bypasses(static_cast<int64_t>(draft->kv.batch) * draft->kv.num_kv_heads * draft->max_budget, FP8);
      span_rows = decode_span_rows(draft->kv, draft->max_budget);
      nspan = (draft->max_budget + span_rows - 1) / span_rows;
      dws = decode_carve(draft->kv, draft->max_budget, draft->workspace);
      n_draft = nspan * draft->kv.num_kv_heads * draft->kv.batch;
    }
    if constexpr (RB <= 2 || (FP8 && RB == 3)) {     // a range per workgroup
      ws.n_ranges = team_ranges(ws.n_ranges);
      if (fused) {
        KernelTimer t("mixed_flash_team", st);
        const auto kernel = may_bypass ? mixed_flash_team<RB, FP8, true> : mixed_flash_team<RB, FP8, false>;
        hipLaunchKernelGGL(kernel, dim3(ws.n_ranges + n_draft), dim3(kTeamWaves * kWave), 0, st, kv, q, a.n_q, ws, out,
                           *draft, dws, span_rows, nspan);
      } else {
        KernelTimer t("verify_flash_team", st);
        // (without the statistic, plain multi-query decode: nothing is stashed, nothing rebuilt)
        const auto kernel = !stats ? verify_flash_team<RB, FP8, kNoStash> : through ? verify_flash_team<RB, FP8, kStashThrough> : verify_flash_team<RB, FP8, kStashKept>;
        hipLaunchKernelGGL(kernel, dim3(ws.n_ranges), dim3(kTeamWaves * kWave), 0, st, kv, q, a.n_q, ws, out);
      }
    } else {                                         // two wavefronts per range and per draft workgroup
      if (fused) {
        KernelTimer t("mixed_flash_pair", st);
        const auto kernel = may_bypass ? mixed_flash_pair<RB, FP8, true> : mixed_flash_pair<RB, FP8, false>;
        hipLaunchKernelGGL(kernel, dim3(ws.n_ranges + n_draft), dim3(2 * kThreads), 0, st, kv, q, a.n_q, ws, out,
                           *draft, dws, span_rows, nspan);
      } else {
        KernelTimer t("verify_flash_pair", st);
        const auto kernel = !stats ? verify_flash_pair<RB, FP8, kNoStash> : through ? verify_flash_pair<RB, FP8, kStashThrough> : verify_flash_pair<RB, FP8, kStashKept>;
        hipLaunchKernelGGL(kernel, dim3(ws.n_ranges), dim3(2 * kThreads), 0, st, kv, q, a.n_q, ws, out);
      }
    }
    int split_select = 0;                      // chunks per row when the selection is a launch of its own
    SelectOut sel{};
    {
      // one workgroup per pair: log-sum-exp, O of split pairs, scores, selection
      KernelTimer t("verify_finish", st);
      sel = a.select ? *a.select : SelectOut{};
#define PILLAR_FINISH(THREADS, CH, SELECT)                                                                                          \
  {                                                                                                                                 \
    const int mergers = merger_groups(pairs, kv.max_seq_len, rows, THREADS, num_cus());                                             \
    if (pairs <= num_cus()) ws.order = nullptr;                                                                                     \
    hipLaunchKernelGGL((verify_finish<RB, THREADS, CH, SELECT, false>), dim3(pairs, mergers + 1), dim3(THREADS), 0, st, kv, a.n_q,  \
                       ws, out, a.lse, a.scores, a.score_stride, sel, mergers);                                                     \
  }
#define PILLAR_FINISH_SPLIT(CH)                                                                                                   \
  {                                                                                                                               \
    const int nchunks = (kv.max_seq_len + 8191) / 8192;                                                                           \
    const int mergers = merger_groups(pairs, kv.max_seq_len, rows, 1024, num_cus());                                              \
    hipLaunchKernelGGL((verify_finish<RB, 1024, 1, false, true>), dim3(pairs, mergers + nchunks), dim3(1024), 0, st, kv, a.n_q,   \
                       ws, out, a.lse, a.scores, a.score_stride, sel, mergers);                                                   \
    split_select = CH;                                                                                                            \
  }
      // few pairs (a unified batch with a handful of verifying requests): every pair gets 16 wavefronts, the
      // kernel then lasts as long as its longest pair; rows beyond 8192 tokens are shared by several workgroups.  Up to two pairs
      // per compute unit, though only one such workgroup is resident: 512 pairs of 4-8 K tokens 42 us (57 when two were
      // resident and merged their segments one by one)
      const bool few = pairs <= 2 * num_cus();
      if (!a.select && a.scores && kv.max_seq_len > 8192 && pairs <= num_cus()) PILLAR_FINISH_SPLIT(0)   // (statistic only)
      else if (!a.select) PILLAR_FINISH(512, 1, false)
      else if (kv.max_seq_len <= 4096 && !few) PILLAR_FINISH(512, 1, true)
      else if (kv.max_seq_len <= 8192 && few) PILLAR_FINISH(1024, 1, true)
      else if (kv.max_seq_len <= 8192) PILLAR_FINISH(512, 2, true)
      // long rows: with fewer pairs than compute units a pair is shared by several workgroups (measured at 128 pairs
      // of 28 K tokens: 121 against 142 us); with more pairs one workgroup per pair keeps everything in one launch
      // (512 pairs of up to 32 K tokens: 149 against 163 us)
      else if (kv.max_seq_len <= 16384 && pairs <= num_cus()) PILLAR_FINISH_SPLIT(2)
      else if (kv.max_seq_len <= 16384) PILLAR_FINISH(1024, 2, true)
      else if (pairs <= num_cus()) PILLAR_FINISH_SPLIT(4)
      else PILLAR_FINISH(1024, 4, true)
#undef PILLAR_FINISH_SPLIT
#undef PILLAR_FINISH
    }
    if (split_select) {
      KernelTimer t("verify_select_rows", st);
      if (split_select == 2) hipLaunchKernelGGL((verify_select_rows<2>), dim3(pairs), dim3(1024), 0, st, kv, ws, a.scores, a.score_stride, sel);
      else hipLaunchKernelGGL((verify_select_rows<4>), dim3(pairs), dim3(1024), 0, st, kv, ws, a.scores, a.score_stride, sel);
    }
    if (fused) {
      const hipError_t e = launch_decode_merge(*draft, st);      // only lists longer than one span leave partials
      if (e != hipSuccess) return e;
    }
    return hipGetLastError();
  }
  {
    KernelTimer t("verify_lse_range", st);
    hipLaunchKernelGGL((verify_lse_range<RB, FP8>), dim3(ws.n_ranges), dim3(kThreads), 0, st, kv, q, a.n_q, ws);
  }
  {
    KernelTimer t("verify_lse_combine", st);
    hipLaunchKernelGGL(verify_lse_combine_range, dim3((pairs * ws.rows_pad + 255) / 256), dim3(256), 0, st, kv, a.n_q, ws, a.lse);
  }
  {
    KernelTimer t("verify_score_range", st);
    hipLaunchKernelGGL((verify_score_range<RB, FP8>), dim3(ws.n_ranges), dim3(kThreads), 0, st, kv, q, a.n_q, ws, out, a.scores,
                       a.score_stride);
  }
  {
    KernelTimer t("verify_o_merge", st);
    hipLaunchKernelGGL(verify_o_merge_range, dim3(pairs), dim3(256), 0, st, kv, a.n_q, ws, out);
  }
  return hipGetLastError();
}

}  // namespace

bool verify_range_supported(const VerifyArgs& a) {
  const KvView& kv = a.kv;
  if (a.q_dtype != PILLAR_BF16) return false;
  if (a.kv_dtype != PILLAR_BF16 && a.kv_dtype != PILLAR_FP8_E4M3) return false;
  if (kv.head_dim != kHeadDim || kv.page_size < 16) return false;
  if (row_blocks(kv, a.n_q) > 4) return false;
  if (!(kv.sm_scale > 0.f)) return false;       // the kernels take row maxima before scaling
  if (a.spec_lens && a.exact_scores) return false;   // per-request lengths: single-pass kernels only
  const int64_t align = a.kv_dtype == PILLAR_BF16 ? 8 : 16;      // elements per 16 bytes
  if (kv.stride_page % align || kv.stride_head % align || kv.stride_slot % align) return false;
  if ((reinterpret_cast<uintptr_t>(kv.k_pool) | reinterpret_cast<uintptr_t>(kv.v_pool) | reinterpret_cast<uintptr_t>(a.q) |
       reinterpret_cast<uintptr_t>(a.out)) & 15u)
    return false;
  // the rows of one load are addressed in 32 bits
  const int64_t esz = a.kv_dtype == PILLAR_BF16 ? 2 : 1, rows = a.kv_dtype == PILLAR_BF16 ? LaneGeom<false>::kRowsPerLoad : LaneGeom<true>::kRowsPerLoad;
  if (kv.stride_slot > ((int64_t{1} << 32) - kHeadDim * esz) / ((rows - 1) * esz)) return false;
  // the statistic is stored four tokens at a time
  if (a.scores && ((reinterpret_cast<uintptr_t>(a.scores) & 15u) || (a.score_stride & 3))) return false;
  // units are counted in 32 bits
  const int64_t units = static_cast<int64_t>(kv.batch) * kv.num_kv_heads * tiles_of_len(kv.max_seq_len);
  return units < (int64_t{1} << 30);
}

bool verify_select_fused(const VerifyArgs& a) {
  // the finish kernel keeps the keys of a row in registers: up to 4 chunks of 8192 tokens; longer rows take the two steps
  return a.select && verify_range_supported(a) && !a.exact_scores && a.kv.max_seq_len <= kFinishMaxTokens;
}

size_t verify_range_workspace(const KvView& kv, int n_q) {
  size_t total = 0;
  carve(kv, n_q, nullptr, &total);
  return total;
}

bool verify_fuses_draft(const VerifyArgs& a) {
  // the fused grid holds the single pass with its statistic and in-kernel selection
  return verify_select_fused(a);
}

hipError_t launch_verify_range(const VerifyArgs& a, hipStream_t s, const DecodeArgs* fused_draft) {
  const int rb = row_blocks(a.kv, a.n_q);
  const bool fp8 = a.kv_dtype == PILLAR_FP8_E4M3;
#define PILLAR_CASE(N) \
  if (rb == N) return fp8 ? run<N, true>(a, s, fused_draft) : run<N, false>(a, s, fused_draft);
  PILLAR_CASE(1)
  PILLAR_CASE(2)
  PILLAR_CASE(3)
  PILLAR_CASE(4)
#undef PILLAR_CASE
  return hipErrorInvalidValue;
}

}  // namespace pillar
