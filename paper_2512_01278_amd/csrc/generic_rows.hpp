// Pieces shared by the kernels for any supported shape and dtype (fp32 arithmetic, the contractions on the matrix cores): K and V rows of a
// 32-token piece are staged in LDS as floats, one element per lane and load, so that lanes read consecutive elements of a
// row whatever its type, stride and alignment, and every element is fetched once per workgroup.
//
// Before, a thread walked a K row by itself (neighbouring lanes a whole row apart) and looked every V row's page up again
// for every element: two requests of 300 and 512 tokens with 16 rows (fp32, head_dim 64)
// took 98 us to verify in three launches (split 70, merge 8, scores 20) and 22.6 to draft from 64 of them, then 24 + 17
// and 9.8, and 9 + 11 with a workgroup per 32 tokens, and 5 + 7 and 6.4 with the contractions on the matrix cores: what is left is the
// chain length -> page -> row -> LDS.
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

// The contractions of a piece on the matrix cores, in fp32 (v_mfma_f32_16x16x4_f32: 16 rows, 16 columns, 4 terms).  With a dot product per
// thread the LDS was what bounded a piece: four multiply-adds of a wavefront took a 16-byte read of K and one of Q, where here 64 do.
// Two fp32 requests of 300 and 512 tokens with 16 rows: split 9.1 -> 5.3 us, finish 10.3 -> 7.0 (query rows and partials are sent for
// earlier as well), draft 9.8 -> 6.4; 16 of 2 K with 64 rows and head_dim 128, whole round 174 -> 83; 256 of 1 K, 2 heads 566 -> 327; 8 of
// 32 K 248 -> 138.  Errors against float64 halved by the four short sums: of the first, outputs 1.1e-6 -> 5.0e-7, scores 3.9e-7 -> 1.6e-7.
typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int kQStride = kGenMaxD + 4;         // floats between staged query rows, as for kPieceStride

// Logits of 16 tokens (block tb of the piece) against 16 query rows (block rb): element i of lane (n, g) is token 16 tb + 4 g + i, row
// 16 rb + n (n = lane % 16, g = lane / 16).  A lane reads four dims at a time and the products take one of each lane group: dims 16 u +
// 4 g + j, g < 4.  Rows past the last give garbage in columns that nobody reads.
template <int D>
__device__ __forceinline__ f32x4 piece_qk(const float* s_rows, const float* s_q, int tb, int rb, int lane) {
  const float* k = s_rows + (16 * tb + (lane & 15)) * kPieceStride + 4 * (lane >> 4);
  const float* q = s_q + (16 * rb + (lane & 15)) * kQStride + 4 * (lane >> 4);
  f32x4 acc[4] = {};                           // four short sums: less rounding than one long one, and no product waits for the last
#pragma unroll
  for (int u = 0; u < D; u += 16) {
    const f32x4 kv = *reinterpret_cast<const f32x4*>(k + u), qv = *reinterpret_cast<const f32x4*>(q + u);
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(kv[j], qv[j], acc[j], 0, 0, 0);
  }
  return (acc[0] + acc[1]) + (acc[2] + acc[3]);
}

// acc += P V of a piece for 16 rows (block rb) and 16 dims (block db): element i of lane (n, g) is row 16 rb + 4 g + i, dim 16 db + n.  p has
// `p_stride` floats per row (a multiple of 4; 4 more than a multiple of 64 or 32 spreads the rows over the banks).  Rows of tokens past
// the end are staged as zeros and their probabilities are zero, so the piece is always walked whole.
__device__ __forceinline__ void piece_pv(const float* s_rows, const float* s_p, int p_stride, int t0, int rb, int db, f32x4& acc, int lane) {
  const float* p = s_p + (16 * rb + (lane & 15)) * p_stride + t0 + 4 * (lane >> 4);
  const float* v = s_rows + 4 * (lane >> 4) * kPieceStride + 16 * db + (lane & 15);
  f32x4 sum[2] = {};
#pragma unroll
  for (int u = 0; u < kPiece; u += 16) {
    const f32x4 pv = *reinterpret_cast<const f32x4*>(p + u);
#pragma unroll
    for (int j = 0; j < 4; ++j) sum[j & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(pv[j], v[(u + j) * kPieceStride], sum[j & 1], 0, 0, 0);
  }
  acc += sum[0] + sum[1];
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

// Softmax of `rows` rows of N logits, `stride` floats apart, in place, relative to the larger of a row's own maximum and floor_of(r): 16 lanes per
// row, 16 rows at a time.  done(r, m, l) is called by one lane per row with the maximum used and the row's sum.
template <int N, int stride, typename Floor, typename Done>
__device__ __forceinline__ void softmax_rows(float* s, int rows, Floor floor_of, Done done) {
  constexpr int kWide = N >= 64 ? 4 : 2, kVecs = N / (16 * kWide);
  typedef float vec __attribute__((ext_vector_type(kWide)));
  const int e = threadIdx.x & 15;
  for (int r = threadIdx.x / 16; r < rows; r += kGenThreads / 16) {
    vec* sr = reinterpret_cast<vec*>(s + r * stride);
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
