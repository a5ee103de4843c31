// The exact integer rate of a bulk flow, floor(bytes * 8000 / duration_ms)
// bit/s saturated to 2^64 - 1, for the classify kernel (kernels.hip) and the
// merge of spilled rows (table.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace gnm {

// floor(b * 8000 / d) for b with 8000*b < 2^53, d >= 1.
constexpr uint64_t kFastBytesMax = ((1ull << 53) - 1ull) / 8000ull;

static __device__ __noinline__ uint64_t rate_bps_wide(uint64_t b, uint32_t d) {
  // floor(8000 b / d) = 8000 floor(b/d) + floor(8000 (b mod d) / d), saturated.
  const uint64_t q1 = b / d, r1 = b % d;
  if (q1 > ~0ull / 8000ull) return ~0ull;
  const uint64_t hi = q1 * 8000ull;
  const uint64_t lo = (r1 * 8000ull) / d;  // r1 * 8000 < 2^45
  const uint64_t s = hi + lo;
  return s < hi ? ~0ull : s;
}

__device__ __forceinline__ uint64_t rate_bps(uint64_t b, uint32_t d) {
  if (b <= kFastBytesMax) {
    const uint64_t num = b * 8000ull;  // < 2^53: exact as a double
    // The correctly rounded quotient is within one of floor(num/d) and never
    // below it; one integer check removes the rounding step up.
    uint64_t q = (uint64_t)((double)num / (double)d);
    const uint64_t prod = q * (uint64_t)d;
    if (prod > num) q -= 1;
    else if (num - prod >= d) q += 1;
    return q;
  }
  return rate_bps_wide(b, d);
}

}  // namespace gnm
