// Sparse draft attention, generic path (any supported shape and dtype, fp32
// arithmetic throughout, the contractions on the matrix cores).
//
// Paper Sections 1 and 4.2: a draft step loads and attends to the critical
// tokens only; with the KV-Cache addressed row by row ("page size 1") this is
// the same pipeline as full attention, driven by an index list.
//
// One workgroup per (request, KV head) walks the index list in tiles of kTile
// rows with a running (max, sum, output): the textbook online softmax.
#include <type_traits>

#include "generic_rows.hpp"
#include "launch.hpp"

namespace pillar {
namespace {

constexpr int kTile = 128, kStride = kTile + 4;
constexpr int kThreads = kGenThreads;
constexpr int kMaxG = 16;

// Workgroups that a compute unit has to hold; what bounds that are the registers of the rows on their way.  The compiler, left to itself, takes
// more for their addresses in the two forms of a tile and holds one workgroup less: 600 (request, head) pairs with lists of 64, head_dim
// 64 and fp32 14.8 us (two per compute unit, 12.8 before the matrix cores) / 10.7 here, bf16 rows 26.9 (19.9) / 16.7, their lists of 1024
// rows 335 (317) / 188; head_dim 128 and fp32, 300 pairs, lists of 64 19.1 (19.6) / 12.2.  The other types do not fit closer without spilling.
constexpr int decode_per_cu(int kvdt, int d) { return d == 64 ? (kvdt == PILLAR_FP8_E4M3 ? 2 : 3) : kvdt == PILLAR_F32 ? 2 : 1; }

template <int QDT, int KVDT, int D>
__global__ __launch_bounds__(kThreads, decode_per_cu(KVDT, D)) void decode_generic(DecodeArgs a) {
  __shared__ __attribute__((aligned(16))) float s_q[kMaxG * kQStride];
  __shared__ __attribute__((aligned(16))) float s[kMaxG * kStride];
  __shared__ __attribute__((aligned(16))) float s_k[kPiece * kPieceStride];
  __shared__ float row_m[kMaxG], row_l[kMaxG], row_alpha[kMaxG];
  __shared__ int64_t s_off[kTile];
  __shared__ float s_ks[kTile], s_vs[kTile];

  const KvView& kv = a.kv;
  const int b = blockIdx.y, g = blockIdx.x;
  const int G = kv.num_q_heads / kv.num_kv_heads;
  const int32_t* list = a.indices + (static_cast<int64_t>(b) * kv.num_kv_heads + g) * a.max_budget;
  int token = list[min(static_cast<int>(threadIdx.x), a.max_budget - 1)];          // (entries up to max_budget exist: no need for the count)
  const int n = min(max(a.counts[b], 0), a.max_budget);

  for (int idx = threadIdx.x; idx < G * D; idx += kThreads)
    s_q[idx / D * kQStride + (idx & (D - 1))] = Storage<QDT>::load(a.q, (static_cast<int64_t>(b) * kv.num_q_heads + g * G) * D + idx);
  if (threadIdx.x < kMaxG) { row_m[threadIdx.x] = -INFINITY; row_l[threadIdx.x] = 0.f; }
  constexpr int kPieces = kTile / kPiece, kDimBlocks = D / 64;
  const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), col = lane & 15, g4 = lane >> 4;
  f32x4 acc[kDimBlocks];                       // element i: row 4 g4 + i, dim 16 (wave + 4 j) + col
#pragma unroll
  for (int j = 0; j < kDimBlocks; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // one tile of nj <= 32 PIECES rows
  auto tile = [&](int j0, int nj, auto count) {
    constexpr int PIECES = decltype(count)::value;
    if (static_cast<int>(threadIdx.x) < nj) {
      int page;
      if (j0 > 0) token = list[j0 + threadIdx.x];
      s_off[threadIdx.x] = row_offset(kv, b, g, token, &page);
      if (KVDT == PILLAR_FP8_E4M3) {
        s_ks[threadIdx.x] = kv.k_scale[static_cast<int64_t>(page) * kv.num_kv_heads + g];
        s_vs[threadIdx.x] = kv.v_scale[static_cast<int64_t>(page) * kv.num_kv_heads + g];
      }
    }
    __syncthreads();
    StagedPiece<KVDT, D> k[PIECES], v[PIECES];         // all rows are sent for before the first is needed
#pragma unroll
    for (int p = 0; p < PIECES; ++p) k[p].fetch(kv.k_pool, s_off, p * kPiece, nj);
#pragma unroll
    for (int p = 0; p < PIECES; ++p) v[p].fetch(kv.v_pool, s_off, p * kPiece, nj);
#pragma unroll
    for (int p = 0; p < kPieces; ++p) {
      const int p0 = p * kPiece, jj = p0 + 16 * (wave & 1) + 4 * g4;
      f32x4 x = {0.f, 0.f, 0.f, 0.f};
      if (p < PIECES && p0 < nj) {             // uniform
        if (p0 > 0) __syncthreads();           // the previous piece has been read
        k[p < PIECES ? p : 0].store(s_k);
        __syncthreads();
        if (wave < 2) x = piece_qk<D>(s_k, s_q, wave, 0, lane);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (KVDT == PILLAR_FP8_E4M3 && jj + i < nj) x[i] *= s_ks[jj + i];
        x[i] = jj + i < nj ? x[i] * kv.sm_scale : -INFINITY;
      }
      if (wave < 2 && col < G) *reinterpret_cast<f32x4*>(s + col * kStride + jj) = x;
    }
    __syncthreads();
    softmax_rows<kTile, kStride>(s, G, [&](int r) { return row_m[r]; }, [&](int r, float m, float l) {      // nj >= 1, so m is finite
      const float alpha = (row_m[r] == -INFINITY) ? 0.f : __expf(row_m[r] - m);
      row_alpha[r] = alpha;
      row_l[r] = row_l[r] * alpha + l;
      row_m[r] = m;
    });
#pragma unroll
    for (int p = 0; p < PIECES; ++p) {
      if (p * kPiece < nj) {                   // uniform
        __syncthreads();                       // the softmax is done; the K rows, or the previous piece, have been read
        if (KVDT == PILLAR_FP8_E4M3) v[p].scale(s_vs, p * kPiece, nj);
        v[p].store(s_k);
        if (p == 0) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float alpha = 4 * g4 + i < G ? row_alpha[4 * g4 + i] : 0.f;
#pragma unroll
            for (int j = 0; j < kDimBlocks; ++j) acc[j][i] *= alpha;
          }
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kDimBlocks; ++j) piece_pv(s_k, s, kStride, p * kPiece, 0, wave + 4 * j, acc[j], lane);
      }
    }
    __syncthreads();
  };
  for (int j0 = 0; j0 < n; j0 += kTile) {
    const int nj = min(kTile, n - j0);
    if (nj <= 2 * kPiece) tile(j0, nj, std::integral_constant<int, 2>{});        // (half the loads and their addresses)
    else tile(j0, nj, std::integral_constant<int, kPieces>{});
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = 4 * g4 + i;
    if (r >= G) continue;
    const int64_t row = static_cast<int64_t>(b) * kv.num_q_heads + g * G + r;
    const float l = row_l[r];
#pragma unroll
    for (int j = 0; j < kDimBlocks; ++j) Storage<QDT>::store(a.out, row * D + 16 * (wave + 4 * j) + col, n > 0 ? acc[j][i] / l : 0.f);
    if (wave == 0 && col == 0 && a.lse) a.lse[row] = n > 0 ? row_m[r] + __logf(l) : -INFINITY;
  }
}

}  // namespace

hipError_t launch_decode_generic(const DecodeArgs& a, hipStream_t s) {
  const dim3 grid(a.kv.num_kv_heads, a.kv.batch);
  KernelTimer t("decode_generic", s);
#define PILLAR_CASE(Q, K)                                                            \
  if (a.q_dtype == Q && a.kv_dtype == K) {                                           \
    if (a.kv.head_dim == 64) hipLaunchKernelGGL((decode_generic<Q, K, 64>), grid, dim3(kThreads), 0, s, a);       \
    else hipLaunchKernelGGL((decode_generic<Q, K, 128>), grid, dim3(kThreads), 0, s, a);                         \
    return hipGetLastError();                                                        \
  }
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
