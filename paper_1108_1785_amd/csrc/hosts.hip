// Per-host rate statistics and medians (§III.B.2, TransRate Kernel: maximum,
// minimum, average and median transfer rates for each host in a registered
// site, the median read from the host's 10 kbps bucket array).
//
// Dense bucket arrays per host do not fit (a 10 M-record window has about
// half a million hosts with bulk flows; 10,001 buckets each would be 21 GB),
// and hash-table updates with device-scope atomics are bound by the rate of
// those atomics.  Here the classify kernel only appends one 16-byte entry
// (host, bytes, duration) per bulk flow of a registered site to its
// workgroup's staging range, and up to four kernels finish the job with no
// per-flow device atomics:
//   1. part_count_kernel: per classify workgroup, the number of its entries
//      in each of P partitions (a partition is the top bits of a hash of the
//      key, so all entries of a host land in one partition); left out where
//      the classify kernel has the LDS to count them as it appends them;
//   2. part_scan_kernel: for each partition, the offset of every workgroup's
//      share within the partition (a column prefix sum) and the totals;
//   3. part_scatter_kernel: every entry to its partition's range;
//   4. host_reduce_kernel: a group of lanes per partition gathers its hosts
//      in an LDS hash map with their statistics (LDS atomics), then finds
//      each host's lower median bucket (the ceil(N/2)-th smallest of its N
//      flows' buckets).  Up to 2,048 entries (nearly every partition): the
//      map has 512 slots, the flow count's atomic gives each flow its place
//      in its host's list, the lists are packed into LDS, and every flow is
//      ranked within its host's list by a lane (of longer lists than 256 a
//      wave finds the median in 7 passes, each leaving a quarter of the
//      range).  More entries (a hot host): a map of 256 slots and a radix
//      selection over the 14-bit bucket, four rounds that read the entries,
//      each counting the candidates' next 4-bit digit in 16 LDS bins per host
//      and keeping the digit where the running count reaches the rank; the
//      first also leaves slot and bucket in the entries for the others.
//      A partition with more hosts than the map holds is done in batches: the
//      entries of hosts not yet in the map are compacted in place and
//      reduced by the next batch.
// Each host is written once, at an index taken from counters[0]; the order
// of hosts therefore depends on timing, the set of (key, statistics, median)
// does not.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <string>

#include "gnm_device.h"
#include "hosts.h"
#include "partition.h"
#include "rate.h"
#include "registry.h"

namespace gnm {

namespace {

constexpr uint32_t kHostThreads = 256;  // lanes that reduce one partition
constexpr uint32_t kHostGroups = 2;     // partitions reduced by one workgroup
constexpr uint32_t kHostSlots = 256;        // LDS hash-map slots of a large partition (a power of two)
constexpr uint32_t kListSlots = 512;        // of one whose flow lists fit LDS: a generated window's mean of 200 to 400
                                            // entries, all of different hosts, must not need a second batch
constexpr uint32_t kListCap = 2048;         // entries of such a partition
constexpr uint32_t kListRank = 256;         // flows of a host that are ranked one against the others
constexpr uint32_t kListSlotBits = 9, kListPlaceBits = 9;
static_assert(kListSlots == 1u << kListSlotBits && kListRank <= 1u << kListPlaceBits, "list words");
constexpr uint64_t kHostEmpty = ~0ull;      // free map slot (no key has all low 32 bits set)
constexpr uint32_t kDigitBins = 16;         // radix selection: 4 bits per round
constexpr uint32_t kDigitRounds = 4;        // buckets < 2^14: digits at bits 12, 8, 4, 0
constexpr uint32_t kPartBitsMin = 6, kPartBitsMax = 14;
constexpr uint32_t kNoSlot = 0xFFFFFFFFu;

typedef u64 u64x2 __attribute__((ext_vector_type(2)));

// Key of an entry's host: remote address << 32 | row.
__device__ __forceinline__ u64 entry_key(u64 x, u64 y, uint32_t vbits) {
  return (x & ~0xFFFFFFFFull) | ((y & ~(u64)kHostWide) >> vbits);
}

// Partition of a host entry: the top pbits of a hash of its key, so all
// entries of a host land in one partition.
struct HostPart {
  uint32_t pbits, vbits;
  static constexpr bool kTotalsHook = false;
  static __device__ __forceinline__ uint32_t part(const HostEntry &e, const HostPart &t) {
    const u64 k = entry_key(e.x, e.y, t.vbits);
    return host_hash((uint32_t)(k >> 32), (uint32_t)k) >> (32u - t.pbits);
  }
};

struct Parts {
  HostEntry *part;
  const uint32_t *ptotal, *pbase;
  u64 *keys, *stats;
  uint32_t *median;
  uint64_t capacity;
  u64 *counters;
  const uint64_t *bytes;  // of the records
  uint32_t vbits;
};

// Bytes and rate of an entry.
__device__ __forceinline__ void entry_rate(const Parts &q, u64x2 e, u64 &bytes, u64 &rate) {
  bytes = e.y & ((1ull << q.vbits) - 1ull);
  if (e.y & kHostWide) bytes = q.bytes[bytes];
  rate = rate_bps(bytes, (uint32_t)e.x);
}

struct HostMap {
  u64 key[kHostSlots];
  u64 bytes[kHostSlots], rsum[kHostSlots], rmin[kHostSlots], rmax[kHostSlots];
  uint32_t flows[kHostSlots];
  uint32_t bins[kDigitBins][kHostSlots];  // digit counts, bin-major so a slot's walk is bank-conflict free
  uint32_t want[kHostSlots];    // rank of the median among the candidates still in play
  uint32_t prefix[kHostSlots];  // digits of the median bucket chosen so far
  uint32_t out[kHostSlots];     // output index of the slot's host within the batch
};

// Slot of key in a map of SLOTS keys, inserting it when absent; kNoSlot when
// the map is full.  Keys are never removed within a batch, so a slot seen
// holding another key stays that way and linear probing needs no locks.
template <uint32_t SLOTS>
__device__ __forceinline__ uint32_t map_insert(u64 *keys, u64 key) {
  uint32_t s = host_hash((uint32_t)(key >> 32), (uint32_t)key) & (SLOTS - 1u);
  for (uint32_t probe = 0; probe < SLOTS; ++probe) {
    u64 cur = keys[s];
    if (cur == kHostEmpty) cur = atomicCAS(&keys[s], kHostEmpty, key);
    if (cur == kHostEmpty || cur == key) return s;
    s = (s + 1u) & (SLOTS - 1u);
  }
  return kNoSlot;
}

template <uint32_t SLOTS>
__device__ __forceinline__ uint32_t map_find(const u64 *keys, u64 key) {
  uint32_t s = host_hash((uint32_t)(key >> 32), (uint32_t)key) & (SLOTS - 1u);
  for (uint32_t probe = 0; probe < SLOTS; ++probe) {
    const u64 cur = keys[s];
    if (cur == key) return s;
    if (cur == kHostEmpty) return kNoSlot;
    s = (s + 1u) & (SLOTS - 1u);
  }
  return kNoSlot;
}

// Choose slot s's next digit: the bin where the running count of its
// candidates reaches its rank (the rank becomes the rank within that bin),
// from the 16 bins read at once; the bins are cleared for the next round.
__device__ __forceinline__ void pick_digit(HostMap &m, uint32_t s) {
  uint32_t b[kDigitBins];
#pragma unroll
  for (uint32_t j = 0; j < kDigitBins; ++j) b[j] = m.bins[j][s];
  const uint32_t want = m.want[s];
  uint32_t c = 0, d = 0, before = 0;
#pragma unroll
  for (uint32_t j = 0; j < kDigitBins - 1u; ++j) {
    c += b[j];
    const bool below = c < want;  // the target lies beyond bin j
    d += below;
    before = below ? c : before;
  }
  m.want[s] = want - before;
  m.prefix[s] = (m.prefix[s] << 4) | d;
#pragma unroll
  for (uint32_t j = 0; j < kDigitBins; ++j) m.bins[j][s] = 0u;
}

constexpr uint32_t kPerThread = 4;  // entries a thread loads before working on them

// The map of a partition of at most kListCap entries.  stat: bytes, rate sum,
// minimum and maximum of each slot's host.
struct ListMap {
  u64 key[kListSlots];
  u64 stat[4][kListSlots];
  uint32_t flows[kListSlots];
  uint16_t base[kListSlots];    // first list element
  uint16_t slot[kListSlots];    // slot of the batch's i-th host
  uint16_t median[kListSlots];  // of each slot's host
  // flows, host by host: bucket << 18 | place among the host's flows (modulo
  // 512) << 9 | slot, so the words of a list of at most 512 are distinct and
  // ordered by bucket
  uint32_t list[kListCap];
  uint16_t queue[kListCap / kListRank];  // slots of longer lists
};

union Maps {
  HostMap big;
  ListMap list;
};

// What the groups of a workgroup share.  Every group takes every barrier, so
// loops around barriers run to the largest n of the workgroup.
struct Shared {
  uint32_t overflow[kHostGroups], deferred[kHostGroups], queued[kHostGroups];
  uint32_t wave[kHostGroups][kHostThreads / 64];
  uint32_t n[kHostGroups];
  u64 out[kHostGroups];
};

// Entries of hosts that found no slot, compacted to the front for the next
// batch: each round reads a block of entries, waits, then writes them at or
// before the block's end, so no entry is overwritten unread.
template <uint32_t SLOTS>
__device__ __forceinline__ void compact_deferred(HostEntry *ent, uint32_t n, uint32_t nmax, const u64 *keys,
                                                 uint32_t vbits, uint32_t *deferred, uint32_t tid) {
  for (uint32_t i0 = 0; i0 < nmax; i0 += kHostThreads) {
    const uint32_t i = i0 + tid;
    u64x2 e{0ull, 0ull};
    bool keep = false;
    if (i < n) {
      e = *(const u64x2 *)(ent + i);
      keep = map_find<SLOTS>(keys, entry_key(e.x, e.y, vbits)) == kNoSlot;
    }
    __syncthreads();
    if (keep) *(u64x2 *)(ent + atomicAdd(deferred, 1u)) = e;
    __syncthreads();
  }
}

// Output indexes for the groups' hosts with one device atomic for the
// workgroup: the atomics of all partitions go to one counter, so each costs
// the chip about 6 ns (4,096 of them took 25 of the kernel's 67 us).
// reserve_out (one thread; sh.wave[g] holds the waves' host counts, in the
// bits from `shift`) starts it, publish_out leaves each group's first index
// in sh.out once its round trip has been covered.
__device__ __forceinline__ u64 reserve_out(const Shared &sh, const Parts &q, uint32_t shift) {
  u64 all = 0;
#pragma unroll
  for (uint32_t g = 0; g < kHostGroups; ++g)
#pragma unroll
    for (uint32_t v = 0; v < kHostThreads / 64u; ++v) all += sh.wave[g][v] >> shift;
  return all ? __hip_atomic_fetch_add(&q.counters[0], all, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0ull;
}

__device__ __forceinline__ void publish_out(Shared &sh, u64 out, uint32_t shift) {
#pragma unroll
  for (uint32_t g = 0; g < kHostGroups; ++g) {
    sh.out[g] = out;
#pragma unroll
    for (uint32_t v = 0; v < kHostThreads / 64u; ++v) out += sh.wave[g][v] >> shift;
  }
}

__device__ __forceinline__ bool any_overflow(const Shared &sh) {
  uint32_t any = 0;
#pragma unroll
  for (uint32_t g = 0; g < kHostGroups; ++g) any |= sh.overflow[g];
  return any != 0u;
}

// One batch of group g's partition of n <= kListCap entries; the entries left
// to the next batch are counted in sh.deferred[g].
__device__ __forceinline__ void reduce_lists(ListMap &m, Shared &sh, const Parts &q, HostEntry *ent, uint32_t n,
                                             uint32_t nmax, uint32_t g) {
  constexpr uint32_t kRounds = kListCap / (kPerThread * kHostThreads);
  const uint32_t tid = threadIdx.x % kHostThreads, lane = tid % 64u, wv = tid / 64u;
  for (uint32_t s = tid; s < kListSlots; s += kHostThreads) {
    m.key[s] = kHostEmpty;
    m.flows[s] = 0u;
    m.stat[0][s] = m.stat[1][s] = m.stat[3][s] = 0;
    m.stat[2][s] = ~0ull;
  }
  if (tid == 0) {
    sh.overflow[g] = 0u;
    sh.deferred[g] = 0u;
    sh.queued[g] = 0u;
  }
  __syncthreads();
  // hosts and statistics; every entry keeps (slot << 14 | bucket) and its
  // place among its host's flows in registers
  uint32_t sb[kRounds * kPerThread], place[kRounds * kPerThread];
#pragma unroll
  for (uint32_t r = 0; r < kRounds; ++r) {
    if (r * kPerThread * kHostThreads >= n) break;
    u64x2 v[kPerThread];
#pragma unroll
    for (uint32_t j = 0; j < kPerThread; ++j) {
      const uint32_t i = (r * kPerThread + j) * kHostThreads + tid;
      if (i < n) v[j] = *(const u64x2 *)(ent + i);
    }
#pragma unroll
    for (uint32_t j = 0; j < kPerThread; ++j) {
      const uint32_t e = r * kPerThread + j, i = e * kHostThreads + tid;
      sb[e] = kNoSlot;
      if (i >= n) continue;
      const uint32_t s = map_insert<kListSlots>(m.key, entry_key(v[j].x, v[j].y, q.vbits));
      if (s == kNoSlot) {
        sh.overflow[g] = 1u;
        continue;
      }
      place[e] = atomicAdd(&m.flows[s], 1u);
      u64 bytes, rate;
      entry_rate(q, v[j], bytes, rate);
      sb[e] = (s << 14) | rate_bucket(rate);
      atomicAdd(&m.stat[0][s], bytes);
      atomicAdd(&m.stat[1][s], rate);
      atomicMin(&m.stat[2][s], rate);
      atomicMax(&m.stat[3][s], rate);
    }
  }
  __syncthreads();
  // slots 2 tid and 2 tid + 1: where their lists start and their places among
  // the batch's hosts (one scan of hosts << 16 | flows)
  static_assert(kListSlots == 2u * kHostThreads, "two slots per thread");
  const uint32_t c0 = m.flows[2u * tid], c1 = m.flows[2u * tid + 1u];
  const uint32_t mine = c0 + c1 + (c0 ? 1u << 16 : 0u) + (c1 ? 1u << 16 : 0u);
  uint32_t x = mine;
#pragma unroll
  for (uint32_t o = 1; o < 64u; o <<= 1) {
    const uint32_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63u) sh.wave[g][wv] = x;
  __syncthreads();
  uint32_t before = x - mine, all = 0;
#pragma unroll
  for (uint32_t v = 0; v < kHostThreads / 64u; ++v) {
    before += v < wv ? sh.wave[g][v] : 0u;
    all += sh.wave[g][v];
  }
  const uint32_t hosts = all >> 16, b0 = before & 0xFFFFu, b1 = b0 + c0;
  const uint32_t h0 = before >> 16, h1 = h0 + (c0 ? 1u : 0u);
  m.base[2u * tid] = (uint16_t)b0;
  m.base[2u * tid + 1u] = (uint16_t)b1;
  if (c0) m.slot[h0] = (uint16_t)(2u * tid);
  if (c1) m.slot[h1] = (uint16_t)(2u * tid + 1u);
  __syncthreads();
  // the batch's output indexes: the round trip overlaps the lists
  u64 first = 0;
  if (threadIdx.x == 0) first = reserve_out(sh, q, 16u);
#pragma unroll
  for (uint32_t e = 0; e < kRounds * kPerThread; ++e) {
    if (e * kHostThreads >= n) break;
    if (e * kHostThreads + tid < n && sb[e] != kNoSlot) {
      const uint32_t sl = sb[e] >> 14, bk = sb[e] & 0x3FFFu;
      m.list[m.base[sl] + place[e]] =
          (bk << (kListSlotBits + kListPlaceBits)) | ((place[e] & ((1u << kListPlaceBits) - 1u)) << kListSlotBits) | sl;
    }
  }
  __syncthreads();
  // lower medians: a lane per flow counts the flows below it in its list; the
  // one with the median's rank writes it.  Neighbouring lanes mostly share a
  // list, so their reads are broadcasts.
  const uint32_t flows = all & 0xFFFFu;
  for (uint32_t i = tid; i < flows; i += kHostThreads) {
    const uint32_t w = m.list[i], sl = w & (kListSlots - 1u);
    const uint32_t c = m.flows[sl], *l = m.list + m.base[sl];
    uint32_t below = 0;
    if (c > kListRank) {
      if (l == m.list + i) m.queue[atomicAdd(&sh.queued[g], 1u)] = (uint16_t)sl;
      continue;
    }
    uint32_t k = 0;
    for (; k + 4u <= c; k += 4u)
      below += (uint32_t)(l[k] < w) + (uint32_t)(l[k + 1u] < w) + (uint32_t)(l[k + 2u] < w) + (uint32_t)(l[k + 3u] < w);
    for (; k < c; ++k) below += l[k] < w;
    if (below + 1u == (c + 1u) / 2u) m.median[sl] = (uint16_t)(w >> (kListSlotBits + kListPlaceBits));
  }
  __syncthreads();
  const uint32_t queued = sh.queued[g];
  for (uint32_t j = wv; j < queued; j += kHostThreads / 64u) {
    // the smallest bucket with at least `want` flows at or below it, a quarter
    // of the range left by each of 7 passes over the list, 8 words of a lane in
    // flight (14 halvings, a word at a time: 20 us more for a list of 700)
    const uint32_t sl = m.queue[j], c = m.flows[sl], base = m.base[sl], want = (c + 1u) / 2u;
    uint32_t lo = 0;
    for (uint32_t q4 = (1u << 14) / 4u; q4; q4 /= 4u) {
      uint32_t below[3] = {0u, 0u, 0u};  // flows below lo + q4, lo + 2 q4, lo + 3 q4
      for (uint32_t k0 = 0; k0 < c; k0 += 8u * 64u) {
        uint32_t v[8];
#pragma unroll
        for (uint32_t i = 0; i < 8u; ++i) {
          const uint32_t k = k0 + i * 64u + lane;
          v[i] = m.list[base + (k < c ? k : 0u)] >> (kListSlotBits + kListPlaceBits) | (k < c ? 0u : 1u << 14);
        }
#pragma unroll
        for (uint32_t i = 0; i < 8u; ++i)
#pragma unroll
          for (uint32_t h = 0; h < 3u; ++h) below[h] += (uint32_t)__popcll(__ballot(v[i] < lo + (h + 1u) * q4));
      }
#pragma unroll
      for (uint32_t h = 3; h > 0u; --h)
        if (below[h - 1u] < want) {
          lo += h * q4;
          break;
        }
    }
    if (lane == 0) m.median[sl] = (uint16_t)lo;
  }
  if (threadIdx.x == 0) publish_out(sh, first, 16u);
  __syncthreads();
  // the batch's hosts, consecutive lanes on consecutive words
  const u64 out = sh.out[g];
  const u64 room = q.capacity > out ? q.capacity - out : 0ull;
  const uint32_t put = hosts < room ? hosts : (uint32_t)room;
  for (uint32_t i = tid; i < put; i += kHostThreads) {
    q.keys[out + i] = m.key[m.slot[i]];
    if (q.median) q.median[out + i] = m.median[m.slot[i]];
  }
  for (uint32_t i = tid; i < 5u * put; i += kHostThreads) {
    const uint32_t h = i / 5u, f = i - 5u * h, s = m.slot[h];
    q.stats[5u * out + i] = f == 0u ? (u64)m.flows[s] : m.stat[f - 1u][s];
  }
  compact_deferred<kListSlots>(ent, sh.overflow[g] ? n : 0u, any_overflow(sh) ? nmax : 0u, m.key, q.vbits,
                               &sh.deferred[g], tid);
}

// One batch of a larger partition (a hot host): every digit round re-reads
// the entries.  The first pass leaves slot << 14 | bucket in place of the
// duration in those that found a slot, so that the rounds need neither the rate
// again (1 M records, half of them one host's: 1,026 us a call with a division
// in every round, 770 now) nor, unless some found none, the map.  A lane always
// reads the same entries.
__device__ __forceinline__ void reduce_radix(HostMap &m, Shared &sh, const Parts &q, HostEntry *ent, uint32_t n,
                                             uint32_t nmax, uint32_t g) {
  static_assert(kHostSlots == kHostThreads, "one map slot per thread");
  const uint32_t tid = threadIdx.x % kHostThreads, lane = tid % 64u, wv = tid / 64u;
  m.key[tid] = kHostEmpty;
  m.flows[tid] = 0u;
  m.bytes[tid] = m.rsum[tid] = m.rmax[tid] = 0;
  m.rmin[tid] = ~0ull;
  m.prefix[tid] = 0u;
#pragma unroll
  for (uint32_t j = 0; j < kDigitBins; ++j) m.bins[j][tid] = 0u;
  if (tid == 0) {
    sh.overflow[g] = 0u;
    sh.deferred[g] = 0u;
  }
  __syncthreads();
  // hosts, statistics and the first digit (bits 13..12) of every bucket;
  // each thread loads kPerThread entries before it works on them
  for (uint32_t i0 = 0; i0 < n; i0 += kPerThread * kHostThreads) {
    u64x2 v[kPerThread];
#pragma unroll
    for (uint32_t j = 0; j < kPerThread; ++j) {
      const uint32_t i = i0 + j * kHostThreads + tid;
      if (i < n) v[j] = *(const u64x2 *)(ent + i);
    }
#pragma unroll
    for (uint32_t j = 0; j < kPerThread; ++j) {
      const uint32_t i = i0 + j * kHostThreads + tid;
      if (i >= n) continue;
      const uint32_t s = map_insert<kHostSlots>(m.key, entry_key(v[j].x, v[j].y, q.vbits));
      if (s == kNoSlot) {
        sh.overflow[g] = 1u;
        continue;
      }
      u64 bytes, rate;
      entry_rate(q, v[j], bytes, rate);
      ent[i].x = (v[j].x & ~0xFFFFFFFFull) | (s << 14) | rate_bucket(rate);
      atomicAdd(&m.flows[s], 1u);
      atomicAdd(&m.bytes[s], bytes);
      atomicAdd(&m.rsum[s], rate);
      atomicMin(&m.rmin[s], rate);
      atomicMax(&m.rmax[s], rate);
      atomicAdd(&m.bins[rate_bucket(rate) >> 12][s], 1u);
    }
  }
  __syncthreads();
  // reserve the batch's output indexes now, so the atomic's round trip
  // overlaps the digit rounds
  const bool used = m.key[tid] != kHostEmpty;
  const u64 bal = __ballot(used);
  if (lane == 0) sh.wave[g][wv] = (uint32_t)__popcll(bal);
  if (used) m.want[tid] = (m.flows[tid] + 1u) / 2u;
  __syncthreads();
  u64 first = 0;
  if (threadIdx.x == 0) first = reserve_out(sh, q, 0u);
  if (used) {
    pick_digit(m, tid);
    uint32_t before = (uint32_t)__popcll(bal & ((1ull << lane) - 1ull));
    for (uint32_t v = 0; v < wv; ++v) before += sh.wave[g][v];
    m.out[tid] = before;
  }
  __syncthreads();
  // the other three digits, among the candidates that share the digits so far
  const bool all = sh.overflow[g] == 0u;
  for (uint32_t r = 1; r < kDigitRounds; ++r) {
    const uint32_t shift = 12u - 4u * r;
    for (uint32_t i0 = 0; i0 < n; i0 += kPerThread * kHostThreads) {
      uint32_t v[kPerThread];
#pragma unroll
      for (uint32_t j = 0; j < kPerThread; ++j) {
        const uint32_t i = i0 + j * kHostThreads + tid;
        v[j] = kNoSlot;
        if (i >= n) continue;
        const u64x2 e = *(const u64x2 *)(ent + i);
        if (all || map_find<kHostSlots>(m.key, entry_key(e.x, e.y, q.vbits)) != kNoSlot) v[j] = (uint32_t)e.x;
      }
#pragma unroll
      for (uint32_t j = 0; j < kPerThread; ++j) {
        if (v[j] == kNoSlot) continue;
        const uint32_t s = v[j] >> 14, bk = v[j] & 0x3FFFu;
        if ((bk >> (shift + 4u)) == m.prefix[s]) atomicAdd(&m.bins[(bk >> shift) & 15u][s], 1u);
      }
    }
    __syncthreads();
    if (used) pick_digit(m, tid);
    __syncthreads();
  }
  if (threadIdx.x == 0) publish_out(sh, first, 0u);
  __syncthreads();
  // write the batch's hosts
  if (used) {
    const uint64_t idx = sh.out[g] + m.out[tid];
    if (idx < q.capacity) {
      q.keys[idx] = m.key[tid];
      u64 *st = q.stats + idx * 5u;
      st[0] = m.flows[tid];
      st[1] = m.bytes[tid];
      st[2] = m.rsum[tid];
      st[3] = m.rmin[tid];
      st[4] = m.rmax[tid];
      if (q.median) q.median[idx] = m.prefix[tid];
    }
  }
  compact_deferred<kHostSlots>(ent, sh.overflow[g] ? n : 0u, any_overflow(sh) ? nmax : 0u, m.key, q.vbits,
                               &sh.deferred[g], tid);
}

// One workgroup per kHostGroups partitions, a group of kHostThreads lanes for
// each.  Small partitions take batches of lists together; large ones then
// batches of the radix selection.
// A window of 10 M records (4,096 partitions of 344 entries, 127 hosts) is
// bound by the latency of a workgroup's steps and by the one counter (entries
// of half the size, as now, changed nothing): 61.7 us with a radix selection for
// every partition; with lists 67 us at one partition per workgroup (42 without
// the counter's atomics), 51.7 at two (50 now), 56 at four (whose barriers wait
// for the slowest of four).  One of 1 M
// records of the 64-site registry (512 partitions of 275 entries, nearly as
// many hosts): 49 us when its hosts overflowed a map of 256 slots, 11.7 now.
__global__ __launch_bounds__(kHostThreads * kHostGroups) void host_reduce_kernel(const Parts q) {
  __shared__ Maps m[kHostGroups];
  __shared__ Shared sh;
  const uint32_t g = threadIdx.x / kHostThreads, p = blockIdx.x * kHostGroups + g;
  HostEntry *ent = q.part + q.pbase[p];
  uint32_t n = q.ptotal[p];
  for (;;) {
    if (threadIdx.x % kHostThreads == 0) sh.n[g] = n;
    __syncthreads();
    uint32_t nlist = 0, nbig = 0;  // largest of either kind
#pragma unroll
    for (uint32_t v = 0; v < kHostGroups; ++v) {
      const uint32_t x = sh.n[v];
      if (x <= kListCap) nlist = x > nlist ? x : nlist;
      else nbig = x > nbig ? x : nbig;
    }
    if (nlist) {
      const uint32_t mine = n <= kListCap ? n : 0u;
      reduce_lists(m[g].list, sh, q, ent, mine, nlist, g);
      __syncthreads();
      if (n <= kListCap) n = sh.deferred[g];
    } else if (nbig) {
      reduce_radix(m[g].big, sh, q, ent, n, nbig, g);
      __syncthreads();
      n = sh.deferred[g];
    } else {
      return;
    }
  }
}

// n == 0: no classify launch and no entries; the counters still start at 0.
__global__ void host_clear_kernel(u64 *counters) {
  counters[0] = 0;
  counters[1] = 0;
}

PartLayout layout(uint64_t n, uint64_t grid) {
  return part_layout(n, grid, 1ull << host_part_bits(n), sizeof(HostEntry));
}

}  // namespace

uint32_t host_part_bits(uint64_t n) {
  // the power of two nearest n / 2048, so 1,448 to 2,896 records a partition:
  // of generated records, 14% of which are such flows, 200 to 400 entries (344
  // of 127 hosts at 10 M records), within the LDS map if every one is of
  // another host
  uint32_t b = kPartBitsMin;
  while (b < kPartBitsMax && (1ull << b) * 2896u <= n) ++b;
  return b;
}

// The size that callers are told, and held to, has room for 32-byte entries:
// twice what the layout takes.
uint64_t host_work_bytes(uint64_t n, uint64_t grid) {
  return part_layout(n, grid, 1ull << host_part_bits(n), 32u).end;
}

HostStage host_stage(void *work, uint64_t n, uint64_t grid) {
  const PartLayout L = layout(n, grid);
  char *w = (char *)work;
  return HostStage{(HostEntry *)(w + L.stage), (uint32_t *)(w + L.scount), (uint32_t *)(w + L.phist),
                   host_part_bits(n)};
}

int host_pipeline_launch(const gnm_host_table *ht, uint64_t n, uint64_t grid, const uint64_t *bytes, uint32_t rows,
                         bool counted, hipStream_t stream) {
  if (n == 0) {
    hipLaunchKernelGGL(host_clear_kernel, dim3(1), dim3(1), 0, stream, (u64 *)ht->counters);
  } else {
    const PartLayout L = layout(n, grid);
    char *w = (char *)ht->work;
    PartArgs<HostEntry> pa{};
    pa.stage = (const HostEntry *)(w + L.stage);
    pa.scount = (const uint32_t *)(w + L.scount);
    pa.n = n;
    pa.grid = (uint32_t)grid;
    const HostPart hp{host_part_bits(n), host_value_bits(rows)};
    pa.nparts = 1u << hp.pbits;
    pa.phist = (uint32_t *)(w + L.phist);
    pa.ptotal = (uint32_t *)(w + L.ptotal);
    pa.pbase = (uint32_t *)(w + L.pbase);
    pa.part = (HostEntry *)(w + L.part);
    pa.staged = (u64 *)ht->counters + 1;
    pa.clear = (u64 *)ht->counters;
    pa.nclear = 2;
    Parts q{};
    q.part = pa.part;
    q.ptotal = pa.ptotal;
    q.pbase = pa.pbase;
    q.keys = (u64 *)ht->keys;
    q.stats = (u64 *)ht->stats;
    q.median = ht->median;
    q.capacity = ht->capacity;
    q.counters = (u64 *)ht->counters;
    q.bytes = bytes;
    q.vbits = hp.vbits;
    const uint32_t P = pa.nparts;
    if (!counted)
      hipLaunchKernelGGL((part_count_kernel<HostEntry, HostPart>), dim3((uint32_t)grid), dim3(kPartThreads), P * 4u,
                         stream, pa, hp);
    hipLaunchKernelGGL((part_scan_kernel<HostEntry, HostPart>), dim3(P / 64u), dim3(64 * kPartScanWaves), 0, stream,
                       pa, hp);
    hipLaunchKernelGGL((part_scatter_kernel<HostEntry, HostPart>), dim3((uint32_t)grid), dim3(kPartThreads),
                       P * 4u, stream, pa, hp);
    static_assert((1u << kPartBitsMin) % kHostGroups == 0, "whole workgroups");
    hipLaunchKernelGGL(host_reduce_kernel, dim3(P / kHostGroups), dim3(kHostThreads * kHostGroups), 0, stream, q);
  }
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    set_last_error(std::string("per-host kernels: ") + hipGetErrorString(e));
    return GNM_E_HIP;
  }
  return GNM_OK;
}

}  // namespace gnm
