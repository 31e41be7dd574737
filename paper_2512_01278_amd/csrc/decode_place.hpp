// Which (request slot, KV head, span) workgroup i of the draft step takes.  Plain arithmetic, also for a host compiler.
#pragma once

#include <cstdint>

namespace pillar {

// Consecutive workgroups run on different XCDs, each with an L2 of its own.  With fp8 the workgroups of one request share the lines its
// page scales lie in, as many as it has rows of its own to fetch, so the heads of a span are given to one XCD: eight requests at a
// time, one per XCD (requests beyond the last multiple of eight are spread as they come).  The place moves on by one XCD from span
// to span and from turn to turn, so that neither a long list nor every eighth request being long loads one XCD alone.
// 64 requests, 8 heads, fp8, in the order of the indices / here: lists of 512 rows (one span) 21.2 / 19.6 us, of 512 beside room for 2048
// 41.0 / 36.8, 5 % of 512 to 32 K tokens 43.5 / 41.1, every eighth list 2048 and the others 64 25.2 / 26.3 (43.0 where a request's spans
// stayed on one XCD, the same one in every turn).
constexpr uint32_t kXcds = 8;

struct DecPlace {
  int slot_b, g, sp;
};

__host__ __device__ inline DecPlace decode_place(bool fp8, uint32_t i, uint32_t batch, uint32_t heads, uint32_t nspan) {
  const uint32_t per = heads * nspan, turn = i / (kXcds * per);
  uint32_t b, r;
  if (fp8 && (turn + 1) * kXcds <= batch) {
    const uint32_t j = i - turn * kXcds * per;
    r = j / kXcds;
    b = turn * kXcds + (j + turn + r % nspan) % kXcds;
  } else {
    b = i / per;
    r = i - b * per;
  }
  DecPlace p;
  p.slot_b = static_cast<int>(b);
  p.g = static_cast<int>(r / nspan);
  p.sp = static_cast<int>(r % nspan);
  return p;
}

}  // namespace pillar
