// Per-host statistics and medians: the interface between the classify
// launcher (kernels.hip) and the per-host kernels (hosts.hip).
//
// The classify kernel appends one entry (host, bytes, duration) per bulk flow
// of a registered site to its workgroup's staging range: workgroup b owns
// entries [lo_b, lo_b + count[b]) of the staging arrays, where [lo_b, hi_b)
// is its slice of the records (a record gives at most one entry, so the range
// always has room).  The per-host kernels then partition the entries by a
// hash of the key and reduce each partition in LDS.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "gnm.h"

namespace gnm {

// One staged bulk flow: one 16-byte word.  The rate and its bucket follow from
// bytes and duration.  `y` holds, from the top, a bit that is set when the
// bytes do not fit, the row (2 * site + direction) from bit `vbits` on, and
// below it the bytes, or the record's index when they do not fit.  `vbits` is
// the launch's: 63 less the bits of a row.  (With 32-byte entries that carried
// rate and bucket too, a 10 M-record window of 1.4 M such flows took 3 us more
// in the classify kernel, which stores them, and 36 us instead of 29 in the
// scatter.)
struct __attribute__((aligned(16))) HostEntry {
  unsigned long long x;  // remote address << 32 | duration in ms
  unsigned long long y;
};
constexpr unsigned long long kHostWide = 1ull << 63;

// Hash of a host: its top bits choose the partition, its low bits the place in
// a partition's map.  Multiplicative hashing in 32 bits: the odd factors are a
// prime near 2^32 times the fraction of the golden ratio, and 2^32 times the
// fractions of the square roots of 3 and 2, with the high half folded into the low one before each, as a product's low
// bits depend on the low bits alone.  (A 64-bit mix of two 64-bit products per
// bulk flow took the classify kernel 123 us on a 10 M-record window, this 107;
// 18.2 and 14.6 on 1 M records of 64 sites.)
__device__ __forceinline__ uint32_t host_hash(uint32_t remote, uint32_t row) {
  uint32_t h = remote + row * 0xBB67AE85u;
  h = (h ^ (h >> 16)) * 0x9E3779B1u;
  h = (h ^ (h >> 15)) * 0x6A09E667u;
  return h ^ (h >> 16);
}

// Bits of a HostEntry's bytes for `rows` rows.  (Rows take at most 30 bits and
// a call with host statistics has fewer than 2^32 records, so that a record's
// index always fits.)
inline uint32_t host_value_bits(uint32_t rows) {
  uint32_t b = 1;
  while (b < 30u && (rows - 1u) >> b) ++b;
  return 63u - b;
}

// Staging arrays written by the classify kernel (device pointers into the
// caller's work buffer).
struct HostStage {
  HostEntry *entry;
  uint32_t *count;  // [grid]: entries staged by each classify workgroup
  uint32_t *phist;  // [grid][2^pbits]: each classify workgroup's entries per partition
  uint32_t pbits;   // partition of an entry: host_hash >> (32 - pbits)
};

// log2 of the partition count for a call over n records: the power of two
// nearest n / 2048, between 2^6 and 2^14.
uint32_t host_part_bits(uint64_t n);

// Bytes of the work buffer for n records on `grid` classify workgroups.
uint64_t host_work_bytes(uint64_t n, uint64_t grid);

// Staging arrays inside a work buffer laid out for (n, grid).
HostStage host_stage(void *work, uint64_t n, uint64_t grid);

// Enqueue the per-host kernels after the classify kernel: partition counts
// (left out when the classify kernel counted its entries per partition and
// cleared ht->counters itself: `counted`), their scan, the scatter into
// partition order and the per-partition reduction into ht's arrays.  With
// n == 0 only the counters are cleared.  bytes: the records' byte counts;
// rows: the table's rows of registered sites.
int host_pipeline_launch(const gnm_host_table *ht, uint64_t n, uint64_t grid, const uint64_t *bytes, uint32_t rows,
                         bool counted, hipStream_t stream);

}  // namespace gnm
