// Pieces shared by the kernels for any supported shape and dtype (fp32 arithmetic on the vector ALUs): K and V rows of a
// 32-token piece are staged in LDS as floats, one element per lane and load, so that lanes read consecutive elements of a
// row whatever its type, stride and alignment, and every element is fetched once per workgroup.
//
// Before, a thread walked a K row by itself (neighbouring lanes a whole row apart) and looked every V row's page up again
// for every element: two requests of 300 and 512 tokens with 16 rows (fp32, head_dim 64)
// took 98 us to verify in three launches (split 70, merge 8, scores 20) and 22.6 to draft from 64 of them, then 24 + 17
// and 9.8, and 9 + 11 with a workgroup per 32 tokens: what is left is the chain length -> page -> row -> LDS.
#pragma once

#include "common.hpp"

namespace pillar {
namespace {

constexpr int kGenThreads = 256;
constexpr int kPiece = 32;                     // tokens staged at a time
constexpr int kPieceRows = kMaxRows / 2;       // query rows a workgroup handles at a time
constexpr int kGenMaxD = 128;
constexpr int kPieceStride = kGenMaxD + 4;     // floats between staged rows: 16-byte reads of neighbouring rows cover all banks

// Rows first .. first + kPiece - 1 of a list of element offsets (LDS) -> registers, coalesced; rows past `count` as zeros.
template <int DT, int D> struct StagedPiece {
  static constexpr int kPerThread = kPiece * D / kGenThreads;
  float v[kPerThread];
  static __device__ __forceinline__ int token(int j) { return (static_cast<int>(threadIdx.x) + j * kGenThreads) / D; }
  __device__ __forceinline__ void fetch(const void* pool, const int64_t* s_off, int first, int count) {
#pragma unroll
    for (int j = 0; j < kPerThread; ++j) {
      const int t = first + token(j);
      v[j] = t < count ? Storage<DT>::load(pool, s_off[t] + (threadIdx.x & (D - 1))) : 0.f;
    }
  }
  __device__ __forceinline__ void scale(const float* s_scale, int first, int count) {
#pragma unroll
    for (int j = 0; j < kPerThread; ++j)
      if (first + token(j) < count) v[j] *= s_scale[first + token(j)];
  }
  __device__ __forceinline__ void store(float* s_rows) const {
#pragma unroll
    for (int j = 0; j < kPerThread; ++j) s_rows[token(j) * kPieceStride + (threadIdx.x & (D - 1))] = v[j];
  }
};

// Dot products of the thread's token (threadIdx.x % 32) with query rows threadIdx.x / 32 + 8 j, j < ROWS / 8 (rows past
// `rows` give garbage that nobody reads), summed over the dimensions in ascending order.
template <int ROWS, int D>
__device__ __forceinline__ void piece_dots(const float* s_rows, const float* s_q, int rows, float (&dot)[ROWS / 8]) {
  const float* kr = s_rows + (threadIdx.x & (kPiece - 1)) * kPieceStride;
  const int r0 = threadIdx.x / kPiece;
#pragma unroll
  for (int j = 0; j < ROWS / 8; ++j) dot[j] = 0.f;
#pragma unroll 4
  for (int d = 0; d < D; d += 4) {
    const float4 k = *reinterpret_cast<const float4*>(kr + d);
#pragma unroll
    for (int j = 0; j < ROWS / 8; ++j) {
      if (8 * j < rows) {                      // uniform
        const float4 q = *reinterpret_cast<const float4*>(s_q + min(r0 + 8 * j, rows - 1) * D + d);
        dot[j] = fmaf(q.x, k.x, dot[j]);
        dot[j] = fmaf(q.y, k.y, dot[j]);
        dot[j] = fmaf(q.z, k.z, dot[j]);
        dot[j] = fmaf(q.w, k.w, dot[j]);
      }
    }
  }
}

// acc[j] += sum over the piece's tokens of p[row][t0 + t] * v[t][d] for the thread's dimension d = threadIdx.x % D and rows
// threadIdx.x / D + (256 / D) j, in ascending order; p has `p_stride` floats per row.  Rows of tokens past the end are staged as
// zeros and their probabilities are zero, so the piece is always walked whole.
template <int ROWS, int D>
__device__ __forceinline__ void piece_pv(const float* s_rows, const float* s_p, int p_stride, int t0, int rows, float (&acc)[ROWS * D / kGenThreads]) {
  constexpr int step = kGenThreads / D;
  const int d = threadIdx.x & (D - 1), r0 = threadIdx.x / D;
#pragma unroll 2
  for (int t = 0; t < kPiece; t += 4) {
    float v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = s_rows[(t + i) * kPieceStride + d];
#pragma unroll
    for (int j = 0; j < ROWS / step; ++j) {
      if (step * j < rows) {                   // uniform
        const float4 p = *reinterpret_cast<const float4*>(s_p + min(r0 + step * j, rows - 1) * p_stride + t0 + t);
        acc[j] = fmaf(p.x, v[0], acc[j]);
        acc[j] = fmaf(p.y, v[1], acc[j]);
        acc[j] = fmaf(p.z, v[2], acc[j]);
        acc[j] = fmaf(p.w, v[3], acc[j]);
      }
    }
  }
}

// maximum / sum over the 16 lanes of a DPP row, in all of them
__device__ __forceinline__ float lanes16_max(float v) {
  v = fmaxf(v, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0xB1, 0xF, 0xF, true)));    // quad_perm [1,0,3,2]
  v = fmaxf(v, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x4E, 0xF, 0xF, true)));    // quad_perm [2,3,0,1]
  v = fmaxf(v, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x141, 0xF, 0xF, true)));   // row_half_mirror
  v = fmaxf(v, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x140, 0xF, 0xF, true)));   // row_mirror
  return v;
}
__device__ __forceinline__ float lanes16_sum(float v) {
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0xB1, 0xF, 0xF, true));
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x4E, 0xF, 0xF, true));
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x141, 0xF, 0xF, true));
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x140, 0xF, 0xF, true));
  return v;
}

// Softmax of `rows` rows of N logits in place, relative to the larger of a row's own maximum and floor_of(r): 16 lanes per
// row, 16 rows at a time.  done(r, m, l) is called by one lane per row with the maximum used and the row's sum.
template <int N, typename Floor, typename Done>
__device__ __forceinline__ void softmax_rows(float* s, int rows, Floor floor_of, Done done) {
  constexpr int kWide = N >= 64 ? 4 : 2, kVecs = N / (16 * kWide);
  typedef float vec __attribute__((ext_vector_type(kWide)));
  const int e = threadIdx.x & 15;
  for (int r = threadIdx.x / 16; r < rows; r += kGenThreads / 16) {
    vec* sr = reinterpret_cast<vec*>(s + r * N);
    vec x[kVecs];
#pragma unroll
    for (int i = 0; i < kVecs; ++i) x[i] = sr[16 * i + e];
    float m = -INFINITY;
#pragma unroll
    for (int i = 0; i < kVecs; ++i)
#pragma unroll
      for (int j = 0; j < kWide; ++j) m = fmaxf(m, x[i][j]);
    m = fmaxf(lanes16_max(m), floor_of(r));
    const float mu = (m == -INFINITY) ? 0.f : m;           // a row that sees no token: exp(-inf) = 0 throughout
    float l = 0.f;
#pragma unroll
    for (int i = 0; i < kVecs; ++i) {
#pragma unroll
      for (int j = 0; j < kWide; ++j) x[i][j] = __expf(x[i][j] - mu);
      sr[16 * i + e] = x[i];
      l += kWide == 2 ? x[i][0] + x[i][1] : (x[i][0] + x[i][1]) + (x[i][kWide - 2] + x[i][kWide - 1]);
    }
    l = lanes16_sum(l);
    if (e == 0) done(r, m, l);
  }
}

}  // namespace
}  // namespace pillar
