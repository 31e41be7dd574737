// The draft step of one (request, KV head, span of the index list) as a device function, shared by the draft
// kernel and by the kernel that runs a unified draft / verify batch in one grid (paper Sections 1 and 4.2).
#pragma once

#include "decode_place.hpp"
#include "host_rules.hpp"
#include "launch.hpp"
#include "mfma_tile.hpp"

namespace pillar {
namespace {

constexpr int kDecWaves = 4;                      // wavefronts per workgroup of the draft kernel
constexpr int kDecThreads = kDecWaves * kWave;

// Resolved rows of two tiles: lane j < 32 holds row j of one tile, lane 32 + j row j of another.
struct Rows {
  uint32_t off16;  // byte offset of the row in a pool, in units of 16 bytes (rows are 16-byte aligned)
  int page;
};

// token position -> page id -> row offset
template <bool FP8>
__device__ __forceinline__ Rows resolve_rows(const KvView& kv, int b, int g, int tok) {
  const int esz = FP8 ? 1 : 2;
  Rows r;
  r.page = kv.block_table[static_cast<int64_t>(b) * kv.block_table_stride + (tok >> kv.page_shift)];
  const int64_t off = (static_cast<int64_t>(r.page) * kv.stride_page + static_cast<int64_t>(g) * kv.stride_head +
                       static_cast<int64_t>(tok & (kv.page_size - 1)) * kv.stride_slot) * esz;
  r.off16 = static_cast<uint32_t>(off >> 4);
  return r;
}

// sends the row loads of the tile whose row offsets half `half` of the lanes (0: lanes 0..31, 1: lanes 32..63) holds; BYPASS: past the Infinity
// Cache
template <bool FP8, bool BYPASS>
__device__ __forceinline__ void issue_rows(const KvView& kv, uint32_t off16, int half, TileRegs<FP8>& t, int lane) {
  constexpr int kRowsPerLoad = FP8 ? 8 : 4;
  constexpr int kLanesPerRow = FP8 ? 8 : 16;
  const int col = (lane % kLanesPerRow) * 16;
  const char* kp = static_cast<const char*>(kv.k_pool);
  const char* vp = static_cast<const char*>(kv.v_pool);
#pragma unroll
  for (int u = 0; u < TileRegs<FP8>::kLoads; ++u) {
    const int row = kRowsPerLoad * u + lane / kLanesPerRow;
    const uint64_t off = (static_cast<uint64_t>(__shfl(off16, 32 * half + row, 64)) << 4) + col;
    const u32x4 *k = reinterpret_cast<const u32x4*>(kp + off), *v = reinterpret_cast<const u32x4*>(vp + off);
    t.k[u] = BYPASS ? __builtin_nontemporal_load(k) : *k;
    t.v[u] = BYPASS ? __builtin_nontemporal_load(v) : *v;
  }
}

// S^T of a tile of fp8 rows, the dims in the order of tile_qk (8 bytes of a row per step), so that a cache of either type that holds the
// same values gives the same bits.  (16 bytes per read would serve two steps, but of other dims: sums in another order.)
__device__ __forceinline__ void tile_qk8(const uint8_t* ktile, const bf16x8 (&qf)[4], f32x4 (&acc)[2][1], int lane) {
  const int n = lane & 15, g = lane >> 4;
#pragma unroll
  for (int sub = 0; sub < 2; ++sub) {
    acc[sub][0] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const u32x2 raw = *reinterpret_cast<const u32x2*>(ktile + (16 * sub + n) * kF8Row + 32 * s + 8 * g);
      acc[sub][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(widen_fp8x8(raw.x, raw.y), qf[s], acc[sub][0], 0, 0, 0);
    }
  }
}

__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
  return f32_to_bf16(a) | (static_cast<uint32_t>(f32_to_bf16(b)) << 16);
}

// The rest of decode_span_body, once the count is known; tok: the index entries of the first round.  (Whole copies for either kind of loads: with
// a branch at the loads 128 requests with lists of 64 to 448 take 34 us, with one around the rounds 29.0, so 28.0.)
template <bool FP8, int WAVES, bool BYPASS>
__device__ __forceinline__ void decode_span_rest(const DecodeArgs& a, const DecWs& ws, int span_rows, int nspan_max, int slot_b, int b, int g, int sp,
                                                 int count, int (&tok)[2], uint8_t (*s_tiles)[kVTileBytes]) {
  const KvView& kv = a.kv;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int n = lane & 15, g4 = lane >> 4;
  const int G = kv.num_q_heads / kv.num_kv_heads;
  uint8_t* s_tile = s_tiles[wave];
  const int32_t* list = a.indices + (static_cast<int64_t>(b) * kv.num_kv_heads + g) * a.max_budget;
  const int j_begin = sp * span_rows;
  uint16_t* out = static_cast<uint16_t*>(a.out);
  auto entry_of = [&](int round, int q) {
    const int tile = wave + WAVES * (4 * round + 2 * q + (lane >> 5));
    return j_begin + tile * kTileTokens + (lane & 31);
  };
  const int j_end = min(count, j_begin + span_rows);
  const int nspan = (count + span_rows - 1) / span_rows;
  const int ntiles = (j_end - j_begin + kTileTokens - 1) / kTileTokens;       // of the span
  const float c2 = kv.sm_scale * kLog2e;

  f32x4 o[1][8];
#pragma unroll
  for (int d = 0; d < 8; ++d) o[0][d] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY, l_run = 0.f;
  if (wave < ntiles) {
    // B operand: lane (n, g4) holds Q[row n][32s + 8 g4 .. +7]
    bf16x8 qf[1][4];
    const uint16_t* qrow = static_cast<const uint16_t*>(a.q) + (static_cast<int64_t>(b) * kv.num_q_heads + g * G + n) * kHeadDim;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      u32x4 v = {0u, 0u, 0u, 0u};
      if (n < G) v = *reinterpret_cast<const u32x4*>(qrow + 32 * s + 8 * g4);
      qf[0][s] = as_bf16x8(v);
    }
    TileRegs<FP8> regs;
    bool first = true;
    for (int round = 0; wave + WAVES * 4 * round < ntiles; ++round) {
      if (round > 0) {
#pragma unroll
        for (int q = 0; q < 2; ++q) tok[q] = list[min(entry_of(round, q), a.max_budget - 1)];
      }
      // one chain for all four tiles: entries -> page ids -> row offsets.  Rows past the end of the list repeat
      // the first row of their tile (masked later); tiles past the end resolve token 0 and are never loaded.
      Rows rr[2];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int head = __shfl(tok[q], lane & 32, 64);
        const int e = entry_of(round, q);
        const bool tile_there = e - (lane & 31) < j_end;
        rr[q] = resolve_rows<FP8>(kv, b, g, e < j_end ? tok[q] : tile_there ? head : 0);
      }
      const int t_first = wave + WAVES * 4 * round;
      issue_rows<FP8, BYPASS>(kv, rr[0].off16, 0, regs, lane);
      float ks0 = 1.f, ks1 = 1.f, vs0 = 1.f, vs1 = 1.f;      // fp8: dequantisation scales of the rows, behind the first tile's rows
      if constexpr (FP8) {
        const int64_t at0 = static_cast<int64_t>(rr[0].page) * kv.num_kv_heads + g, at1 = static_cast<int64_t>(rr[1].page) * kv.num_kv_heads + g;
        ks0 = kv.k_scale[at0];
        vs0 = kv.v_scale[at0];
        ks1 = kv.k_scale[at1];
        vs1 = kv.v_scale[at1];
      }
      for (int k = 0; k < 4; ++k) {
        const int ti = t_first + WAVES * k;
        if (ti >= ntiles) break;
        const int jb = j_begin + ti * kTileTokens;
        const float k_scale = (k & 2) ? ks1 : ks0, v_scale = (k & 2) ? vs1 : vs0;
        const int half = k & 1;
        const bool more = k < 3 && ti + WAVES < ntiles;
        f32x4 s[2][1];
        if constexpr (FP8) {                     // both tiles have room, as they are
          rows8_to_lds(regs.k, s_tile, lane);
          rows8_to_lds(regs.v, s_tile + kF8TileBytes, lane);
        } else {
          rows_to_lds<false, false>(regs.k, s_tile, lane);
          tile_qk<1>(s_tile, qf, s, lane);
          rows_to_lds<false, true>(regs.v, s_tile, lane);
        }
        if (more) issue_rows<FP8, BYPASS>(kv, ((k + 1) & 2) ? rr[1].off16 : rr[0].off16, (k + 1) & 1, regs, lane);
        if constexpr (FP8) tile_qk8(s_tile, qf[0], s, lane);
        f32x4 vsc[2];
#pragma unroll
        for (int sub = 0; sub < 2; ++sub) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int slot = 16 * sub + 4 * g4 + i;
            float sc = c2;
            vsc[sub][i] = 1.f;
            if constexpr (FP8) {
              sc *= __shfl(k_scale, 32 * half + slot, 64);
              vsc[sub][i] = __shfl(v_scale, 32 * half + slot, 64);
            }
            float v = s[sub][0][i] * sc;
            if (jb + slot >= j_end) v = -INFINITY;
            s[sub][0][i] = v;
          }
        }
        float mx = fmaxf(fmaxf(fmaxf(s[0][0][0], s[0][0][1]), fmaxf(s[0][0][2], s[0][0][3])),
                         fmaxf(fmaxf(s[1][0][0], s[1][0][1]), fmaxf(s[1][0][2], s[1][0][3])));
        mx = max_over_groups(mx);
        const float m_new = fmaxf(m_run, mx);              // finite: every tile has a valid row
        // (exp2f, not the bare instruction, which takes weights below 2^-126 for zero: the values they weigh may be large.  Costs 0.2 us
        // of 19.5 at 64 requests with fp8 lists of 512, 0.3 of 32.0 at 128 with bf16 lists of 64 to 448.)
        const float alpha = exp2f(m_run - m_new);
        f32x4 p0, p1;
        float sum = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          p0[i] = exp2f(s[0][0][i] - m_new);
          p1[i] = exp2f(s[1][0][i] - m_new);
          sum += p0[i] + p1[i];
        }
        l_run = l_run * alpha + sum;
        m_run = m_new;
        if (!first) {
#pragma unroll
          for (int d = 0; d < 8; ++d) o[0][d] *= alpha;
        }
        first = false;
        if constexpr (FP8) { p0 *= vsc[0]; p1 *= vsc[1]; }
        bf16x8 p[1];
        p[0] = pack_p(p0, p1);
        if constexpr (FP8) tile_pv8<1>(s_tile + kF8TileBytes, p, o, lane);
        else tile_pv<1>(s_tile, p, o, lane);
      }
    }
    l_run = sum_over_groups(l_run);
  }

  // combine the wavefronts of the workgroup: every one leaves (max, sum) per row and its O rows in its own tile
  // buffer (a wavefront that had no tile leaves max = -inf, sum = 0)
  float* part = reinterpret_cast<float*>(s_tile);          // [G][128] O, then [16] max, [16] sum
  if (n < G) {
#pragma unroll
    for (int db = 0; db < 8; ++db) *reinterpret_cast<f32x4*>(part + n * kHeadDim + 16 * db + 4 * g4) = o[0][db];
    if (g4 == 0) { part[16 * kHeadDim + n] = m_run; part[16 * kHeadDim + 16 + n] = l_run; }
  }
  __syncthreads();
  for (int idx = threadIdx.x; idx < G * (kHeadDim / 4); idx += (WAVES * kWave)) {
    const int r = idx / (kHeadDim / 4), d4 = idx - r * (kHeadDim / 4);
    float m = -INFINITY;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) m = fmaxf(m, reinterpret_cast<const float*>(s_tiles[w])[16 * kHeadDim + r]);
    float l = 0.f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
      const float* pw = reinterpret_cast<const float*>(s_tiles[w]);
      const float wgt = exp2f(pw[16 * kHeadDim + r] - m);        // m is finite: the first wavefront always has a tile
      l = fmaf(pw[16 * kHeadDim + 16 + r], wgt, l);
      acc += *reinterpret_cast<const f32x4*>(pw + r * kHeadDim + 4 * d4) * wgt;
    }
    const int64_t row = static_cast<int64_t>(b) * kv.num_q_heads + g * G + r;
    if (nspan == 1) {
      const float inv = 1.0f / l;
      u32x2 pk;
      pk.x = pack_bf16x2(acc.x * inv, acc.y * inv);
      pk.y = pack_bf16x2(acc.z * inv, acc.w * inv);
      *reinterpret_cast<u32x2*>(out + row * kHeadDim + 4 * d4) = pk;
      if (d4 == 0 && a.lse) a.lse[row] = (m + log2f(l)) * kLn2;
    } else {
      const int64_t slot = (static_cast<int64_t>(slot_b) * kv.num_kv_heads + g) * nspan_max + sp;
      if (d4 == 0) { ws.part_m[slot * 16 + r] = m; ws.part_l[slot * 16 + r] = l; }
      *reinterpret_cast<f32x4*>(ws.part_o + (slot * G + r) * kHeadDim + 4 * d4) = acc;
    }
  }
}

// One (request slot, KV head, span) of the draft step by a workgroup of WAVES wavefronts.  s_tiles: per
// wavefront one tile buffer (the K rows, then, once S^T is done, the V rows of the same tile; at the end its
// (max, sum, O) for the combine).  MAY_BYPASS: the index buffers have room for so many rows that they might bypass the Infinity Cache; a
// workgroup decides by its own list.  Every thread of the workgroup must call this.
template <bool FP8, int WAVES, bool MAY_BYPASS>
__device__ __forceinline__ void decode_span_body(const DecodeArgs& a, const DecWs& ws, int span_rows, int nspan_max, int slot_b, int g,
                                                 int sp, uint8_t (*s_tiles)[kVTileBytes]) {
  const KvView& kv = a.kv;
  const int b = request_of(kv, slot_b);          // everything the request owns is indexed by its id
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int G = kv.num_q_heads / kv.num_kv_heads;
  const int32_t* list = a.indices + (static_cast<int64_t>(b) * kv.num_kv_heads + g) * a.max_budget;
  const int j_begin = sp * span_rows;
  // The index entries of the first four tiles of this wavefront (tiles wave, wave + WAVES, ...; register q holds
  // tile 2q in lanes 0..31 and tile 2q + 1 in lanes 32..63) leave together with the count: entries up to
  // max_budget exist, which of them count is decided when both are here.
  auto entry_of = [&](int round, int q) {
    const int tile = wave + WAVES * (4 * round + 2 * q + (lane >> 5));
    return j_begin + tile * kTileTokens + (lane & 31);
  };
  int tok[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) tok[q] = list[min(entry_of(0, q), a.max_budget - 1)];
  const int count = min(max(a.counts[b], 0), a.max_budget);
  uint16_t* out = static_cast<uint16_t*>(a.out);
  if (count == 0) {
    if (sp == 0) {
      for (int idx = threadIdx.x; idx < G * kHeadDim; idx += (WAVES * kWave))
        out[(static_cast<int64_t>(b) * kv.num_q_heads + g * G) * kHeadDim + idx] = 0;
      if (a.lse && threadIdx.x < G) a.lse[static_cast<int64_t>(b) * kv.num_q_heads + g * G + threadIdx.x] = -INFINITY;
    }
    return;
  }
  if (j_begin >= count) return;
  if (MAY_BYPASS && draft_bypasses(static_cast<int64_t>(count) * kv.batch * kv.num_kv_heads, FP8))
    decode_span_rest<FP8, WAVES, true>(a, ws, span_rows, nspan_max, slot_b, b, g, sp, count, tok, s_tiles);
  else
    decode_span_rest<FP8, WAVES, false>(a, ws, span_rows, nspan_max, slot_b, b, g, sp, count, tok, s_tiles);
}

}  // namespace
}  // namespace pillar
