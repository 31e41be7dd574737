// Verification attention, generic path: any supported shape and dtype, fp32
// arithmetic throughout (vector ALUs, and fp32 matrix instructions for the
// contractions).  It serves the shapes the bf16 matrix-core path does not
// cover (fp32 tensors, head_dim 64) and is the in-library cross-check of it.
//
// Paper Section 4.1: the k+1 verification rows attend to the whole KV-Cache;
// the softmax probabilities, averaged over those rows and the query heads of
// one GQA group, are the score statistic that Top-K later reads.
//
// Two or three launches:
//   split   one workgroup per (request, KV head, chunk of 128 or 32 tokens):
//           logits of all R=(k+1)*G rows against the chunk, chunk-local
//           softmax, partial output -> workspace
//   merge   (contexts of more than kInlineChunks chunks) one workgroup per
//           (request, KV head, row): log-sum-exp and output from the partials
//   finish  same grid as split: (up to kInlineChunks chunks) log-sum-exp of
//           every row from the partials, and a share of the output; then
//           logits again, now against the final lse: exp(s - lse) is the exact
//           softmax probability; mean over rows
#include <algorithm>
#include <type_traits>

#include "generic_rows.hpp"
#include "launch.hpp"

namespace pillar {
namespace {

// Tokens per workgroup.  The pieces of 32 tokens of a chunk follow each other through LDS, with two barriers and a walk over the
// rows each, so a launch is as long as its longest chunk until the chip is full: up to 4 pieces per compute unit, what the LDS is room for
// (head_dim 128: the split kernel has registers for 3), every piece is a chunk.  Chunks of 128 / of 32 tokens, verification and
// selection and draft, fp32, 4 heads, head_dim 64: 2 requests of 300 to 512 tokens 32.2 / 25.0 us, 4 of 2 K and 2 heads 35.9 / 30.0; 1024
// pieces: 64 of 512 33.5 / 31.7, 16 of 2 K 38.1 / 33.9, 32 of 1 K 34.1 / 35.4; with head_dim 128 49.9 / 48.2, 53.3 / 50.1, 49.5 / 52.0, with fp8
// 116 / 88, 128 / 108, 113 / 92.  Beyond, chunks of 128 fetch the query rows and leave partial outputs a quarter as often.  (The host knows no
// lengths: it counts with max_seq_len, so a caller whose contexts are short does well to say so.)
constexpr int kChunk = 128, kFineChunk = kPiece;
size_t fine_chunks() { return 4 * static_cast<size_t>(num_cus()); }
constexpr int kThreads = kGenThreads;

// Without a merge launch every workgroup of the finish kernel reads the (m, l) of all chunks: quadratic in the context.  With
// one of its own / without, fp32, whole round: 2 requests of 300 to 512 tokens 27.7 / 25.0 us, 64 of 512 34.7 / 31.9, 256 of 1 K with 2 heads
// 348 / 327.  Before the matrix cores: 8 of 2048 179 / 184, 8 of 32 K 2416 / 4666, one of 2 M tokens 2.7 / 139 ms (with one
// workgroup per (request, KV head) instead of one per row: 101).
constexpr int kInlineChunks = 8;

struct GenericWs {
  float* part_m;   // [B][Hkv][NC][R]
  float* part_l;   // [B][Hkv][NC][R]     (merged: the rows' log-sum-exp in chunk 0's place)
  float* part_o;   // [B][Hkv][NC][R][D]
  int nc;
  bool fine;       // chunks of kFineChunk tokens
  bool merged;     // a launch of its own merges (NC > kInlineChunks)
};

__host__ __device__ inline int num_chunks(int max_seq_len) { return (max_seq_len + kChunk - 1) / kChunk; }

template <int CHUNK> struct GenericLds {
  static constexpr int kStride = CHUNK + 4;
  __attribute__((aligned(16))) float q[kPieceRows * kQStride];       // query rows at work
  __attribute__((aligned(16))) float s[kPieceRows * kStride];        // their logits, then probabilities
  __attribute__((aligned(16))) float rows[kPiece * kPieceStride];    // K or V rows of a piece
  int64_t off[CHUNK];                                                // element offset of every token's row
  float ks[CHUNK], vs[CHUNK];                                        // fp8: scales of its page
  float lse[kMaxRows];
};

template <int KVDT, int CHUNK>
__device__ __forceinline__ void resolve_chunk(const KvView& kv, int b, int g, int t0, int nt, GenericLds<CHUNK>& lds) {
  for (int tt = threadIdx.x; tt < nt; tt += kThreads) {
    int page;
    lds.off[tt] = row_offset(kv, b, g, t0 + tt, &page);
    if (KVDT == PILLAR_FP8_E4M3) {
      lds.ks[tt] = kv.k_scale[static_cast<int64_t>(page) * kv.num_kv_heads + g];
      lds.vs[tt] = kv.v_scale[static_cast<int64_t>(page) * kv.num_kv_heads + g];
    }
  }
}

// Up to kPieceRows query rows on their way to LDS, all sent for at once (a loop of loads and stores waits for memory in every turn: of the
// 9 us that two requests of 300 to 512 tokens took to split, 3; so did the last half of the finish kernel).
template <int QDT, int D> struct StagedQueries {
  static constexpr int kPerThread = kPieceRows * D / kThreads;
  float v[kPerThread];
  __device__ __forceinline__ void fetch(const KvView& kv, const void* q, int n_q, int b, int g, int row0, int rows) {
    const int G = kv.num_q_heads / kv.num_kv_heads, inv_g = ((1 << 16) + G - 1) / G;         // r / G: exact for r < 64, G <= 16
#pragma unroll
    for (int j = 0; j < kPerThread; ++j) {
      const int idx = static_cast<int>(threadIdx.x) + j * kThreads, r = row0 + idx / D, i = (r * inv_g) >> 16;
      v[j] = idx < rows * D ? Storage<QDT>::load(q, ((static_cast<int64_t>(b) * n_q + i) * kv.num_q_heads + g * G + r - i * G) * D + (idx & (D - 1))) : 0.f;
    }
  }
  __device__ __forceinline__ void store(float* s_q, int rows) const {
#pragma unroll
    for (int j = 0; j < kPerThread; ++j) {
      const int idx = static_cast<int>(threadIdx.x) + j * kThreads;
      if (idx < rows * D) s_q[idx / D * kQStride + (idx & (D - 1))] = v[j];
    }
  }
};

// Logits of query rows row0 .. row0+rows-1 against the chunk's tokens into lds.s[r][tt] (sm_scale applied, -inf where masked or
// beyond the sequence).  Every thread of the workgroup calls this; lds.off is complete (a barrier ago).
// All K rows are sent for before the first is needed (SENT: they have been, into `sent`), and `ahead` is called right after (to send for
// V rows).  QUERIES_SENT: the query rows are on their way as well (`queries`); a full chip has nothing to gain from that, nor the registers.
template <int QDT, int KVDT, int D, int CHUNK, bool SENT, bool QUERIES_SENT, typename Ahead>
__device__ __forceinline__ void chunk_logits(const KvView& kv, const void* q, int n_q, int b, int g, int t0, int nt, int L, int row0, int rows,
                                             GenericLds<CHUNK>& lds, const StagedPiece<KVDT, D> (&sent)[CHUNK / kPiece],
                                             const StagedQueries<QDT, D>& queries, Ahead ahead) {
  constexpr int kPieces = CHUNK / kPiece;
  StagedPiece<KVDT, D> piece[kPieces];
#pragma unroll
  for (int p = 0; p < kPieces; ++p) {
    if constexpr (SENT) piece[p] = sent[p];
    else piece[p].fetch(kv.k_pool, lds.off, p * kPiece, nt);
  }
  ahead();
  const int G = kv.num_q_heads / kv.num_kv_heads;
  if constexpr (QUERIES_SENT) {
    queries.store(lds.q, rows);
  } else {
    for (int idx = threadIdx.x; idx < rows * D; idx += kThreads) {
      const int r = row0 + idx / D, d = idx & (D - 1);
      const int i = r / G, hg = r - i * G;
      lds.q[(r - row0) * kQStride + d] = Storage<QDT>::load(q, ((static_cast<int64_t>(b) * n_q + i) * kv.num_q_heads + g * G + hg) * D + d);
    }
  }
  // a wavefront takes 16 tokens of a piece against 16 rows
  const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), tb = wave & 1, rb = wave >> 1;
  const int r = 16 * rb + (lane & 15), inv_g = ((1 << 16) + G - 1) / G;
  const int last = L - n_q + (((row0 + r) * inv_g) >> 16);             // the row's last token
#pragma unroll
  for (int p = 0; p < kPieces; ++p) {
    const int p0 = p * kPiece;
    f32x4 x = {0.f, 0.f, 0.f, 0.f};
    if (p0 < nt) {                             // uniform
      __syncthreads();                         // the previous piece has been read
      piece[p].store(lds.rows);
      __syncthreads();
      if (16 * rb < rows) x = piece_qk<D>(lds.rows, lds.q, tb, rb, lane);
    }
    const int tt = p0 + 16 * tb + 4 * (lane >> 4);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (KVDT == PILLAR_FP8_E4M3 && tt + i < nt) x[i] *= lds.ks[tt + i];
      x[i] = t0 + tt + i < L && t0 + tt + i <= last ? x[i] * kv.sm_scale : -INFINITY;
    }
    if (r < rows) *reinterpret_cast<f32x4*>(lds.s + r * GenericLds<CHUNK>::kStride + tt) = x;
  }
  __syncthreads();
}

// (Fine chunks with head_dim 128: the query rows that are sent for early leave registers for three workgroups per compute unit.  With fp8 the
// compiler, left to itself, took enough for two: 48 requests of 512 tokens, this kernel 37.3 us, 23.4 with three, 31.4 before the matrix cores.)
template <int QDT, int KVDT, int D, int CHUNK>
__global__ __launch_bounds__(kThreads, CHUNK == kFineChunk ? (D == 64 ? 4 : 3) : 2) void verify_split_generic(KvView kv, const void* q, int n_q, GenericWs ws) {
  constexpr int kPieces = CHUNK / kPiece;
  __shared__ GenericLds<CHUNK> lds;
  const int b = blockIdx.z, g = blockIdx.y, c = blockIdx.x;
  const int L = kv.seq_lens[b];
  const int t0 = c * CHUNK;
  const int G = kv.num_q_heads / kv.num_kv_heads;
  const int R = n_q * G;
  StagedQueries<QDT, D> queries;
  if constexpr (CHUNK == kFineChunk) queries.fetch(kv, q, n_q, b, g, 0, min(kPieceRows, R));
  if (t0 >= L) return;
  const int nt = min(CHUNK, L - t0);
  const int64_t slot = (static_cast<int64_t>(b) * kv.num_kv_heads + g) * ws.nc + c;
  resolve_chunk<KVDT>(kv, b, g, t0, nt, lds);
  __syncthreads();
  for (int row0 = 0; row0 < R; row0 += kPieceRows) {
    const int rows = min(kPieceRows, R - row0);
    if constexpr (CHUNK == kFineChunk) {
      if (row0 > 0) queries.fetch(kv, q, n_q, b, g, row0, rows);
    }
    StagedPiece<KVDT, D> piece[kPieces];
    chunk_logits<QDT, KVDT, D, CHUNK, false, CHUNK == kFineChunk>(kv, q, n_q, b, g, t0, nt, L, row0, rows, lds, piece, queries, [&]() {
#pragma unroll
      for (int p = 0; p < kPieces; ++p) piece[p].fetch(kv.v_pool, lds.off, p * kPiece, nt);
    });
    softmax_rows<CHUNK, GenericLds<CHUNK>::kStride>(lds.s, rows, [](int) { return -INFINITY; }, [&](int r, float m, float l) {
      ws.part_m[slot * R + row0 + r] = m;
      ws.part_l[slot * R + row0 + r] = l;
    });
    // a wavefront takes every fourth block of 16 dims
    constexpr int kRowBlocks = kPieceRows / 16, kDimBlocks = D / 64;
    const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    f32x4 acc[kRowBlocks][kDimBlocks];
#pragma unroll
    for (int rb = 0; rb < kRowBlocks; ++rb)
#pragma unroll
      for (int j = 0; j < kDimBlocks; ++j) acc[rb][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int p = 0; p < kPieces; ++p) {
      if (p * kPiece < nt) {                   // uniform
        __syncthreads();                       // the K rows, or the previous piece, have been read; the softmax is done
        if (KVDT == PILLAR_FP8_E4M3) piece[p].scale(lds.vs, p * kPiece, nt);
        piece[p].store(lds.rows);
        __syncthreads();
#pragma unroll
        for (int rb = 0; rb < kRowBlocks; ++rb) {
          if (16 * rb < rows) {                // uniform
#pragma unroll
            for (int j = 0; j < kDimBlocks; ++j) piece_pv(lds.rows, lds.s, GenericLds<CHUNK>::kStride, p * kPiece, rb, wave + 4 * j, acc[rb][j], lane);
          }
        }
      }
    }
#pragma unroll
    for (int rb = 0; rb < kRowBlocks; ++rb) {
#pragma unroll
      for (int j = 0; j < kDimBlocks; ++j) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int r = 16 * rb + 4 * (lane >> 4) + i;
          if (r < rows) ws.part_o[(slot * R + row0 + r) * D + 16 * (wave + 4 * j) + (lane & 15)] = acc[rb][j][i];
        }
      }
    }
    __syncthreads();                           // before the next rows' logits
  }
}

// log-sum-exp of a row with maximum m and sum l; a row that sees no token at all (l = 0) has +inf, no weight in the statistic,
// and the caller gets -inf
__device__ __forceinline__ float row_lse(float m, float l) { return l > 0.f ? m + __logf(l) : INFINITY; }
__device__ __forceinline__ float lse_for_caller(float v) { return v == INFINITY ? -INFINITY : v; }

// Chunks are taken in turn by kParts groups of D threads, a dimension per thread.
constexpr int kMergeThreads = 1024;
template <int QDT, int D>
__global__ __launch_bounds__(kMergeThreads) void verify_merge_generic(KvView kv, int n_q, GenericWs ws, void* out, float* lse_out) {
  constexpr int kParts = kMergeThreads / D, kWaves = kMergeThreads / kWave;
  __shared__ float s_m[kWaves], s_l[kWaves], s_o[kMergeThreads];
  const int b = blockIdx.z, g = blockIdx.y, r = blockIdx.x;
  const int G = kv.num_q_heads / kv.num_kv_heads;
  const int R = n_q * G;
  const int chunk = ws.fine ? kFineChunk : kChunk, nc = (max(kv.seq_lens[b], 0) + chunk - 1) / chunk;
  const int64_t base = ((static_cast<int64_t>(b) * kv.num_kv_heads + g) * ws.nc) * R + r;      // (m, l) of chunk 0; R floats from chunk to chunk
  const int wave = threadIdx.x / kWave, lane = threadIdx.x & (kWave - 1);
  float m = -INFINITY;
#pragma unroll 4
  for (int i = threadIdx.x; i < nc; i += kMergeThreads) m = fmaxf(m, ws.part_m[base + static_cast<int64_t>(i) * R]);
  m = wave_max(m);
  if (lane == 0) s_m[wave] = m;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kWaves; ++w) m = fmaxf(m, s_m[w]);
  auto weight = [&](float mc) { return mc == -INFINITY ? 0.f : __expf(mc - m); };
  float l = 0.f;
#pragma unroll 4
  for (int i = threadIdx.x; i < nc; i += kMergeThreads) l = fmaf(ws.part_l[base + static_cast<int64_t>(i) * R], weight(ws.part_m[base + static_cast<int64_t>(i) * R]), l);
  l = wave_sum(l);
  if (lane == 0) s_l[wave] = l;
  const int d = threadIdx.x & (D - 1);
  float o = 0.f;
#pragma unroll 4
  for (int i = threadIdx.x / D; i < nc; i += kParts) {
    const int64_t at = base + static_cast<int64_t>(i) * R;
    o = fmaf(ws.part_o[at * D + d], weight(ws.part_m[at]), o);
  }
  s_o[threadIdx.x] = o;
  __syncthreads();
  if (threadIdx.x >= D) return;
  l = 0.f;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) l += s_l[w];
#pragma unroll
  for (int p = 1; p < kParts; ++p) o += s_o[p * D + d];
  const int i = r / G, hg = r - i * G;
  const int64_t row = (static_cast<int64_t>(b) * n_q + i) * kv.num_q_heads + g * G + hg;
  Storage<QDT>::store(out, row * D + d, l > 0.f ? o / l : 0.f);
  if (d == 0) {
    const float v = row_lse(m, l);
    ws.part_l[base] = v;                       // (read before the last barrier by the threads that needed it)
    if (lse_out) lse_out[row] = lse_for_caller(v);
  }
}

// Workgroups of the finish kernel of fine chunks that a compute unit holds (registers; the LDS is room for four).  EARLY: what is needed
// after the log-sum-exp, the query rows and the partials of 16 chunks instead of 8, is sent for before it.  With head_dim 128 that takes 165
// registers, with fp8 199, so it is for launches that fit on the chip that way.  Whole rounds without / with it, fp32, 4 heads, head_dim
// 128: 2 requests of 300 to 512 tokens and 32 rows 36.7 / 34.7 us, 8 of 2 K and 64 rows 57.4 / 52.5, 48 of 512 41.3 / 39.1; 64 of 512, which do
// not fit, 48.3 / 50.3, with fp8 88.3 / 98.7, 32 of 1 K 92.5 / 106.  (8: of a pair's up to 32 chunks as many as four workgroups leave
// registers for.  16: of two requests of 512 tokens all.)
constexpr int finish_per_cu(int kvdt, int d, bool early) { return d == 64 || !early ? 4 : kvdt == PILLAR_FP8_E4M3 ? 2 : 3; }

template <int QDT, int KVDT, int D, int CHUNK, bool MERGED, bool EARLY>
__global__ __launch_bounds__(kThreads, CHUNK == kFineChunk ? finish_per_cu(KVDT, D, EARLY) : 2) void verify_finish_generic(
    KvView kv, const void* q, int n_q, GenericWs ws, void* out, float* lse_out, float* scores, int64_t score_stride) {
  __shared__ GenericLds<CHUNK> lds;
  const int b = blockIdx.z, g = blockIdx.y, c = blockIdx.x;
  const int L = kv.seq_lens[b];
  const int t0 = c * CHUNK;
  const int G = kv.num_q_heads / kv.num_kv_heads;
  const int R = n_q * G;
  if (t0 >= L) {
    if (!MERGED && c == 0) {                   // an empty context: no query sees a token
      for (int idx = threadIdx.x; idx < R * D; idx += kThreads) {
        const int r = idx / D, i = r / G, hg = r - i * G;
        const int64_t row = (static_cast<int64_t>(b) * n_q + i) * kv.num_q_heads + g * G + hg;
        Storage<QDT>::store(out, row * D + (idx & (D - 1)), 0.f);
        if (lse_out && (idx & (D - 1)) == 0) lse_out[row] = -INFINITY;
      }
    }
    return;
  }
  const int nc = (L + CHUNK - 1) / CHUNK;
  const int nt = min(CHUNK, L - t0);
  const int64_t base = (static_cast<int64_t>(b) * kv.num_kv_heads + g) * ws.nc;
  // A fine chunk's K rows are on their way while the partials are merged.  (Where the chip is full there is nothing to wait for, and
  // rows held that long cost: 64 requests of 1 to 2 K tokens, 64 rows, head_dim 128, this kernel 136 -> 148 us before the matrix cores.)
  constexpr bool kSent = CHUNK == kFineChunk, kQueriesSent = kSent && EARLY;
  StagedQueries<QDT, D> queries;
  if constexpr (kQueriesSent) {
    if (scores) queries.fetch(kv, q, n_q, b, g, 0, min(kPieceRows, R));
  }
  // and so are the partials of this thread's first element of the output
  constexpr int kAhead = kSent && !MERGED ? (EARLY ? 16 : 8) : 1;
  float m_ahead[kAhead], o_ahead[kAhead];
  if constexpr (kAhead > 1) {
    const int idx = min(c * R * D / nc + static_cast<int>(threadIdx.x), R * D - 1);
#pragma unroll
    for (int i = 0; i < kAhead; ++i) {
      const int64_t at = (base + min(i, nc - 1)) * R + idx / D;
      m_ahead[i] = ws.part_m[at];
      o_ahead[i] = ws.part_o[at * D + (idx & (D - 1))];
    }
  }
  StagedPiece<KVDT, D> k_piece[CHUNK / kPiece];
  if (scores) {                                // uniform
    resolve_chunk<KVDT>(kv, b, g, t0, nt, lds);
    if constexpr (kSent) {
      __syncthreads();
#pragma unroll
      for (int p = 0; p < CHUNK / kPiece; ++p) k_piece[p].fetch(kv.k_pool, lds.off, p * kPiece, nt);
    }
  }
  if constexpr (MERGED) {
    if (threadIdx.x < R) lds.lse[threadIdx.x] = ws.part_l[base * R + threadIdx.x];
  } else {                                     // log-sum-exp of every row: four threads per row take the chunks in turn
    const int r = threadIdx.x / 4, part = threadIdx.x & 3;
    constexpr int kMine = kInlineChunks * (kChunk / CHUNK) / 4;          // chunks of a thread, sent for side by side
    float mc[kMine], lc[kMine], m = -INFINITY, l = 0.f;
#pragma unroll
    for (int i = 0; i < kMine; ++i) {
      const int64_t at = (base + min(part + 4 * i, nc - 1)) * R + min(r, R - 1);
      mc[i] = ws.part_m[at];
      lc[i] = ws.part_l[at];
    }
#pragma unroll
    for (int i = 0; i < kMine; ++i) {
      if (part + 4 * i >= nc) mc[i] = -INFINITY;
      m = fmaxf(m, mc[i]);
    }
    m = fmaxf(m, __shfl_xor(m, 1, kWave));
    m = fmaxf(m, __shfl_xor(m, 2, kWave));
#pragma unroll
    for (int i = 0; i < kMine; ++i)
      if (mc[i] != -INFINITY) l = fmaf(lc[i], __expf(mc[i] - m), l);
    l += __shfl_xor(l, 1, kWave);
    l += __shfl_xor(l, 2, kWave);
    if (r < R && part == 0) {
      const float v = row_lse(m, l);
      lds.lse[r] = v;
      if (c == 0 && lse_out) {
        const int i = r / G, hg = r - i * G;
        lse_out[(static_cast<int64_t>(b) * n_q + i) * kv.num_q_heads + g * G + hg] = lse_for_caller(v);
      }
      lds.q[r] = m;                            // for the weights of the output (the query rows come later)
      lds.q[kMaxRows + r] = l > 0.f ? l : 0.f;
    }
    __syncthreads();
    // this workgroup's share of the output
    for (int idx = c * R * D / nc + threadIdx.x; idx < (c + 1) * R * D / nc; idx += kThreads) {      // (few chunks: 32 bits are enough)
      const int r = idx / D, d = idx & (D - 1);
      float o = 0.f;
      auto add = [&](float mc, float po) {
        const float w = (mc == -INFINITY) ? 0.f : __expf(mc - lds.q[r]);
        o = fmaf(po, w, o);
      };
      int i0 = 0;
      if constexpr (kAhead > 1) {
        if (idx < c * R * D / nc + kThreads) {               // the thread's first
#pragma unroll
          for (int i = 0; i < kAhead; ++i)
            if (i < nc) add(m_ahead[i], o_ahead[i]);
          i0 = kAhead;
        }
      }
#pragma unroll 8
      for (int i = i0; i < nc; ++i) add(ws.part_m[(base + i) * R + r], ws.part_o[((base + i) * R + r) * D + d]);
      const int i = r / G, hg = r - i * G;
      Storage<QDT>::store(out, ((static_cast<int64_t>(b) * n_q + i) * kv.num_q_heads + g * G + hg) * D + d,
                          lds.q[kMaxRows + r] > 0.f ? o / lds.q[kMaxRows + r] : 0.f);
    }
  }
  if (!scores) return;
  __syncthreads();                             // the query rows take the place of the weights
  const float inv_r = 1.0f / static_cast<float>(R);
  constexpr int kPer = kThreads / CHUNK;
  float sum = 0.f;                             // of this thread's token
  for (int row0 = 0; row0 < R; row0 += kPieceRows) {
    const int rows = min(kPieceRows, R - row0);
    if constexpr (kSent) {
      if (row0 > 0) {
#pragma unroll
        for (int p = 0; p < CHUNK / kPiece; ++p) k_piece[p].fetch(kv.k_pool, lds.off, p * kPiece, nt);
        if constexpr (kQueriesSent) queries.fetch(kv, q, n_q, b, g, row0, rows);
      }
    }
    chunk_logits<QDT, KVDT, D, CHUNK, kSent, kQueriesSent>(kv, q, n_q, b, g, t0, nt, L, row0, rows, lds, k_piece, queries, []() {});
    // kPer threads per token take the rows in turn
    const int tt = threadIdx.x / kPer;
#pragma unroll 4
    for (int r = threadIdx.x % kPer; r < rows; r += kPer) {
      const float v = lds.s[r * GenericLds<CHUNK>::kStride + tt];
      sum += (v == -INFINITY) ? 0.f : __expf(v - lds.lse[row0 + r]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int o = 1; o < kPer; o <<= 1) sum += __shfl_xor(sum, o, kWave);
  const int tt = threadIdx.x / kPer;
  if (threadIdx.x % kPer == 0 && tt < nt) scores[(static_cast<int64_t>(b) * kv.num_kv_heads + g) * score_stride + t0 + tt] = sum * inv_r;
}

// (request, KV head, chunk) slots of the workspace.  With room for fine chunks: as many as either chunk size takes, so that a smaller
// batch or a shorter context never needs more.
size_t chunk_slots(const KvView& kv, bool fine_room) {
  const size_t n = static_cast<size_t>(kv.batch) * kv.num_kv_heads * num_chunks(kv.max_seq_len);
  return fine_room ? std::max<size_t>(n, kChunk / kFineChunk * std::min<size_t>(n, fine_chunks() * kFineChunk / kChunk)) : n;
}

GenericWs carve(const KvView& kv, int n_q, void* workspace, bool fine_room) {
  const int G = kv.num_q_heads / kv.num_kv_heads;
  const size_t R = static_cast<size_t>(n_q) * G;
  const size_t nc = num_chunks(kv.max_seq_len);
  const size_t slots = chunk_slots(kv, fine_room);
  char* p = static_cast<char*>(workspace);
  GenericWs w;
  w.merged = nc > kInlineChunks;
  w.fine = fine_room && static_cast<size_t>(kv.batch) * kv.num_kv_heads * nc * (kChunk / kFineChunk) <= fine_chunks();
  w.nc = w.fine ? (kv.max_seq_len + kFineChunk - 1) / kFineChunk : static_cast<int>(nc);
  w.part_m = reinterpret_cast<float*>(p); p += align_up(slots * R * 4, 256);
  w.part_l = reinterpret_cast<float*>(p); p += align_up(slots * R * 4, 256);
  w.part_o = reinterpret_cast<float*>(p);
  return w;
}

template <int QDT, int KVDT, int D>
hipError_t run(const VerifyArgs& a, hipStream_t st) {
  const KvView& kv = a.kv;
  const GenericWs ws = carve(kv, a.n_q, a.workspace, a.fine_room);
  const dim3 grid(ws.nc, kv.num_kv_heads, kv.batch);
  {
    KernelTimer t("verify_split_generic", st);
    const auto kernel = ws.fine ? verify_split_generic<QDT, KVDT, D, kFineChunk> : verify_split_generic<QDT, KVDT, D, kChunk>;
    hipLaunchKernelGGL(kernel, grid, dim3(kThreads), 0, st, kv, a.q, a.n_q, ws);
  }
  if (ws.merged) {
    KernelTimer t("verify_merge_generic", st);
    const int R = a.n_q * (kv.num_q_heads / kv.num_kv_heads);
    hipLaunchKernelGGL((verify_merge_generic<QDT, D>), dim3(R, kv.num_kv_heads, kv.batch), dim3(kMergeThreads), 0, st, kv, a.n_q, ws, a.out, a.lse);
  }
  if (!ws.merged || a.scores) {
    KernelTimer t("verify_finish_generic", st);
    const bool early = static_cast<size_t>(grid.x) * grid.y * grid.z <= finish_per_cu(KVDT, D, true) * static_cast<size_t>(num_cus());
    const auto form = [&](auto chunk, auto sent) {
      constexpr int CHUNK = decltype(chunk)::value;
      constexpr bool EARLY = decltype(sent)::value;
      return ws.merged ? verify_finish_generic<QDT, KVDT, D, CHUNK, true, EARLY> : verify_finish_generic<QDT, KVDT, D, CHUNK, false, EARLY>;
    };
    const std::integral_constant<int, kFineChunk> fine{};
    // (head_dim 64: any fine launch fits)
    const auto kernel = !ws.fine ? form(std::integral_constant<int, kChunk>{}, std::false_type{})
                        : early ? form(fine, std::true_type{}) : form(fine, std::bool_constant<D == 64>{});
    hipLaunchKernelGGL(kernel, grid, dim3(kThreads), 0, st, kv, a.q, a.n_q, ws, a.out, a.lse, a.scores, a.score_stride);
  }
  return hipGetLastError();
}

}  // namespace

size_t verify_generic_workspace(const KvView& kv, int n_q, bool fine_room) {
  const size_t R = static_cast<size_t>(n_q) * (kv.num_q_heads / kv.num_kv_heads), slots = chunk_slots(kv, fine_room);
  return 2 * align_up(slots * R * 4, 256) + align_up(slots * R * kv.head_dim * 4, 256);
}

hipError_t launch_verify_generic(const VerifyArgs& a, hipStream_t s) {
#define PILLAR_CASE(Q, K) \
  if (a.q_dtype == Q && a.kv_dtype == K) return a.kv.head_dim == 64 ? run<Q, K, 64>(a, s) : run<Q, K, 128>(a, s);
  PILLAR_CASE(PILLAR_F32, PILLAR_F32)
  PILLAR_CASE(PILLAR_F32, PILLAR_BF16)
  PILLAR_CASE(PILLAR_F32, PILLAR_FP8_E4M3)
  PILLAR_CASE(PILLAR_BF16, PILLAR_F32)
  PILLAR_CASE(PILLAR_BF16, PILLAR_BF16)
  PILLAR_CASE(PILLAR_BF16, PILLAR_FP8_E4M3)
#undef PILLAR_CASE
  return hipErrorInvalidValue;
}

}  // namespace pillar
