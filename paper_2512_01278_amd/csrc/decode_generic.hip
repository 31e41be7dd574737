// Sparse draft attention, generic path (any supported shape and dtype, fp32
// arithmetic on the vector ALUs).
//
// Paper Sections 1 and 4.2: a draft step loads and attends to the critical
// tokens only; with the KV-Cache addressed row by row ("page size 1") this is
// the same pipeline as full attention, driven by an index list.
//
// One workgroup per (request, KV head) walks the index list in tiles of kTile
// rows with a running (max, sum, output): the textbook online softmax.
#include "generic_rows.hpp"
#include "launch.hpp"

namespace pillar {
namespace {

constexpr int kTile = 128;
constexpr int kThreads = kGenThreads;
constexpr int kMaxG = 16;

template <int QDT, int KVDT, int D>
__global__ __launch_bounds__(kThreads) void decode_generic(DecodeArgs a) {
  __shared__ __attribute__((aligned(16))) float s_q[kMaxG * kGenMaxD];
  __shared__ __attribute__((aligned(16))) float s[kMaxG * kTile];
  __shared__ __attribute__((aligned(16))) float s_k[kPiece * kPieceStride];
  __shared__ float row_m[kMaxG], row_l[kMaxG], row_alpha[kMaxG];
  __shared__ int64_t s_off[kTile];
  __shared__ float s_ks[kTile], s_vs[kTile];

  const KvView& kv = a.kv;
  const int b = blockIdx.y, g = blockIdx.x;
  const int G = kv.num_q_heads / kv.num_kv_heads;
  const int n = min(max(a.counts[b], 0), a.max_budget);
  const int32_t* list = a.indices + (static_cast<int64_t>(b) * kv.num_kv_heads + g) * a.max_budget;

  for (int idx = threadIdx.x; idx < G * D; idx += kThreads)
    s_q[idx] = Storage<QDT>::load(a.q, (static_cast<int64_t>(b) * kv.num_q_heads + g * G) * D + idx);
  if (threadIdx.x < kMaxG) { row_m[threadIdx.x] = -INFINITY; row_l[threadIdx.x] = 0.f; }
  constexpr int step = kThreads / D, kPieces = kTile / kPiece;
  float acc[kMaxG / step];                     // dimension threadIdx.x % D of rows threadIdx.x / D + step * j
#pragma unroll
  for (int j = 0; j < kMaxG / step; ++j) acc[j] = 0.f;

  for (int j0 = 0; j0 < n; j0 += kTile) {
    const int nj = min(kTile, n - j0);
    if (static_cast<int>(threadIdx.x) < nj) {
      int page;
      s_off[threadIdx.x] = row_offset(kv, b, g, list[j0 + threadIdx.x], &page);
      if (KVDT == PILLAR_FP8_E4M3) {
        s_ks[threadIdx.x] = kv.k_scale[static_cast<int64_t>(page) * kv.num_kv_heads + g];
        s_vs[threadIdx.x] = kv.v_scale[static_cast<int64_t>(page) * kv.num_kv_heads + g];
      }
    }
    __syncthreads();
    StagedPiece<KVDT, D> k[kPieces], v[kPieces];       // all rows are sent for before the first is needed
#pragma unroll
    for (int p = 0; p < kPieces; ++p) k[p].fetch(kv.k_pool, s_off, p * kPiece, nj);
#pragma unroll
    for (int p = 0; p < kPieces; ++p) v[p].fetch(kv.v_pool, s_off, p * kPiece, nj);
#pragma unroll
    for (int p = 0; p < kPieces; ++p) {
      const int p0 = p * kPiece;
      float dot[kMaxG / 8];
      if (p0 < nj) {                           // uniform
        if (p0 > 0) __syncthreads();           // the previous piece has been read
        k[p].store(s_k);
        __syncthreads();
        piece_dots<kMaxG, D>(s_k, s_q, G, dot);
      }
      const int jj = p0 + (threadIdx.x & (kPiece - 1));
#pragma unroll
      for (int j = 0; j < kMaxG / 8; ++j) {
        const int r = threadIdx.x / kPiece + 8 * j;
        if (r < G) {
          float x = -INFINITY;
          if (jj < nj) {
            x = dot[j];
            if (KVDT == PILLAR_FP8_E4M3) x *= s_ks[jj];
            x *= kv.sm_scale;
          }
          s[r * kTile + jj] = x;
        }
      }
    }
    __syncthreads();
    softmax_rows<kTile>(s, G, [&](int r) { return row_m[r]; }, [&](int r, float m, float l) {      // nj >= 1, so m is finite
      const float alpha = (row_m[r] == -INFINITY) ? 0.f : __expf(row_m[r] - m);
      row_alpha[r] = alpha;
      row_l[r] = row_l[r] * alpha + l;
      row_m[r] = m;
    });
#pragma unroll
    for (int p = 0; p < kPieces; ++p) {
      if (p * kPiece < nj) {                   // uniform
        __syncthreads();                       // the softmax is done; the K rows, or the previous piece, have been read
        if (KVDT == PILLAR_FP8_E4M3) v[p].scale(s_vs, p * kPiece, nj);
        v[p].store(s_k);
        if (p == 0) {
#pragma unroll
          for (int j = 0; j < kMaxG / step; ++j) {
            const int r = threadIdx.x / D + step * j;
            if (r < G) acc[j] *= row_alpha[r];
          }
        }
        __syncthreads();
        piece_pv<kMaxG, D>(s_k, s, kTile, p * kPiece, G, acc);
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int j = 0; j < kMaxG / step; ++j) {
    const int r = threadIdx.x / D + step * j, d = threadIdx.x & (D - 1);
    if (r < G) {
      const int64_t row = static_cast<int64_t>(b) * kv.num_q_heads + g * G + r;
      const float l = row_l[r];
      Storage<QDT>::store(a.out, row * D + d, n > 0 ? acc[j] / l : 0.f);
      if (d == 0 && a.lse) a.lse[row] = n > 0 ? row_m[r] + __logf(l) : -INFINITY;
    }
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
