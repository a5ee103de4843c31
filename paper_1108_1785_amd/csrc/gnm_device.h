// Device helpers shared by the classify kernels (kernels.hip), the histogram
// kernels (hist.hip) and the per-host statistics kernels (hosts.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace gnm {

typedef unsigned long long u64;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr uint32_t kBuckets = 10001;  // rate histogram: 10 kbps buckets, the last for >= 100 Mbps
constexpr uint32_t kBucketBps = 10000;
constexpr uint32_t kXcds = 8;  // workgroups are dealt to these round robin; each has its own L2

// First record of classify workgroup b's slice of n records on `grid`
// workgroups: an even split cut at multiples of 4 records (slice `grid`
// starts at n, where the last one ends).
__host__ __device__ inline uint64_t slice_lo(uint32_t b, uint64_t n, uint32_t grid) {
  return b < grid ? ((uint64_t)b * n / grid) & ~3ull : n;
}

// Classify workgroup whose share of a partition is the i-th: by XCD (b mod 8,
// as workgroups are dealt), so that the scatter workgroups of an XCD fill
// neighbouring entries and its L2 writes whole lines back: 1.4 M 16-byte
// entries scattered in 24 us, in the order of b in 29; 4-byte keys 12.6 and
// 13.2.  0 for i >= grid, a scan wave without a share (below 8 workgroups there
// is nothing to divide by).
__host__ __device__ inline uint32_t part_source(uint32_t i, uint32_t grid) {
  if (i >= grid) return 0u;
  const uint32_t per = grid / kXcds, longer = (grid % kXcds) * (per + 1u);  // the first XCDs have one more
  if (i < longer) return (i % (per + 1u)) * kXcds + i / (per + 1u);
  const uint32_t j = i - longer;
  return (j % per) * kXcds + grid % kXcds + j / per;
}

__host__ __device__ inline uint32_t part_next_source(uint32_t b, uint32_t grid) {
  return b + kXcds < grid ? b + kXcds : b % kXcds + 1u;
}

// Histogram bucket of a rate (§III.B.2, TransRate Kernel): floor(rate /
// 10 kbps), every rate of 100 Mbps and above in the last bucket.
__device__ __forceinline__ uint32_t rate_bucket(uint64_t rate) {
  constexpr uint64_t kTop = (uint64_t)kBucketBps * (kBuckets - 1u);  // 100 Mbps
  return rate >= kTop ? kBuckets - 1u : (uint32_t)rate / kBucketBps;
}

}  // namespace gnm
