// Merge of spilled accumulator rows (§III.B.2, TransRate Kernel: per-site
// statistics; here for registries whose table does not fit LDS).
//
// The classify kernel stages the rows that miss its LDS row cache, and the
// cached rows it flushes at window changes, as 16-byte entries that lie by tile
// of table rows in every workgroup's range, in parts of one size and, for tiles
// whose part is full, in chunks (see table.h).  table_reduce_kernel gives each
// (window, tile) one workgroup, which owns those rows: it sums the entries of
// its tile and window, from the part and chunks of every classify workgroup
// whose slice meets the window, in an LDS table (one LDS atomic per field),
// adds them into its rows of the device table (initialised before the classify
// kernel unless the call accumulates, and holding whatever a workgroup added
// there with device atomics because its range had no room) and applies the
// mean-rate flag test to the sites of its rows.  Device-scope atomics run at
// about 23 G/s on MI355X.
// A tile of many entries (neighbouring sites that are in use) is shared by
// further workgroups, which add their sums to the device table with atomics;
// the last of them applies the flag test.
// What bounds it: a classify workgroup's cache requests (a read of the trie
// for most records, and 16 bytes stored per entry: the store costs a request
// whether it lands in L2 or beyond, and gathering a wave's entries in LDS
// before storing them changed nothing, 1,289 against 1,296 us).  Entries of 32
// bytes in the order they came, ordered by three partition kernels (counts,
// scan, scatter) that read and wrote all of them twice more, took 1,179 + 131
// + 5 + 447 + 184 us for 10 windows of 10 M records and 20,000 sites; lying by
// tile as they are written they took 1,289 + 144 us (24-byte entries, two
// stores each: 1,335 + 193), now 1,251 + 100.  Tiles of 512 or 1,024 rows (fewer, denser parts)
// gain 5 to 10 % there and lose 8 to 25 % on one window, whose merge then has
// too few workgroups.
// With parts alone, what did not fit went to device atomics.  One window of 10 M
// records by the sites in use, us a call: ordered by partition kernels, by tile
// in parts alone, and in parts and chunks with shared tiles:
//   20,000 sites, 500 neighbours      263    291   112
//                 2,000               778    667   233
//                 all, evenly         619    270   237
//                 Zipf, in order      636    454   195
//   1,000,000     2,000               824  1,772   420
//                 20,000              692  2,247   602
//                 all, evenly         880    961   506
//                 Zipf, in order      896  1,185   521
#include <hip/hip_runtime.h>

#include <cstdint>
#include <mutex>
#include <string>

#include "gnm_device.h"
#include "partition.h"
#include "rate.h"
#include "registry.h"
#include "table.h"

namespace gnm {

namespace {

constexpr uint32_t kTableThreads = 1024;
constexpr uint32_t kRowWords = 9;         // u64 words from one LDS row to the next: 8 and a bank pair of padding
constexpr uint32_t kSplitEntries = 8192;  // entries of a tile for each workgroup beyond its own
constexpr int kWaitVmem = 0x0F70;         // s_waitcnt vmcnt(0), the other counters left alone

struct Merge {
  const char *entry;
  const uint32_t *count, *hot;
  uint32_t *done;
  const uint64_t *woff;  // NULL: one window
  uint64_t n, extra;
  uint32_t grid;
  u64 *acc;
  uint32_t rows, tiles, tile_bits, n_windows;
  uint32_t more;  // workgroups per window beyond one per tile
  BulkRule bulk;
  TableFlags fl;
};

typedef u64 u64x2 __attribute__((ext_vector_type(2)));

// First of the part's n entries whose window is at least w (windows ascend).
__device__ __forceinline__ uint32_t first_of_window(const TableEntry *e, uint32_t n, uint32_t w, uint32_t shift) {
  uint32_t lo = 0, len = n;
  while (len) {
    const uint32_t half = len / 2u;
    if ((uint32_t)(e[lo + half].y >> shift) < w) {
      lo += half + 1u;
      len -= half + 1u;
    } else {
      len = half;
    }
  }
  return lo;
}

__device__ __forceinline__ uint64_t readlane64(uint64_t x, uint32_t l) {
  return (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), l) << 32 |
         (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, l);
}

// Workgroups beyond its own that share a tile of `hot` entries over all windows
// (of `all` in all tiles): one for every kSplitEntries per window, or as many
// more as keeps the sum over tiles within q.more.
__device__ __forceinline__ uint32_t split_of(const Merge &q, uint32_t hot, uint32_t all) {
  const uint32_t least = kSplitEntries * q.n_windows, fit = all / q.more + 1u;
  return hot / (least > fit ? least : fit);
}

// What the merge looks up of a classify workgroup: its slice, the entries that a
// part of its range holds, and those that the tile's has.
struct Looked {
  uint64_t lo, hi;
  uint32_t cap, in;
};

// Sum of `hot` over the tiles (every lane takes part; s: a word per wave).
__device__ __forceinline__ uint32_t sum_hot(const Merge &q, uint32_t *s) {
  uint32_t x = 0;
  for (uint32_t j = threadIdx.x; j < q.tiles; j += kTableThreads) x += q.hot[j];
#pragma unroll
  for (uint32_t o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  __syncthreads();
  if (threadIdx.x % 64u == 0u) s[threadIdx.x / 64u] = x;
  __syncthreads();
  x = 0;
#pragma unroll
  for (uint32_t v = 0; v < kTableThreads / 64u; ++v) x += s[v];
  return x;
}

// floor(a * b / c) for a * b < 2^52 and a quotient that is no closer below a
// whole number than 2^-32 (c < 2^32) where it is below 2^20, or than 2^-20 (c <
// 2^20) where it is below 2^32: a double's rounding stays on its side.
__device__ __forceinline__ uint64_t scaled(uint64_t a, uint64_t b, uint64_t c) {
  return (uint64_t)((double)(a * b) / (double)c);
}

// slice_lo of a spilled call, which has fewer than 2^32 records and 2^20 workgroups.
__device__ __forceinline__ uint64_t part_lo(const Merge &q, uint32_t b) {
  return b < q.grid ? scaled(b, q.n, q.grid) & ~3ull : q.n;
}

// Mean-rate test of the registered sites whose rows lie among the nr from r0 on
// of window w; `rows`: those rows, `stride` words apart.
__device__ __forceinline__ void flag_rows(const Merge &q, uint32_t w, uint32_t r0, uint32_t nr, const u64 *rows,
                                          uint32_t stride) {
  for (uint32_t j = threadIdx.x; 2u * j < nr; j += kTableThreads) {
    const uint32_t site = r0 / 2u + j;
    if (site >= q.fl.n_sites) continue;
    uint8_t fv = 0;
#pragma unroll
    for (uint32_t d = 0; d < 2u; ++d) {
      const u64 nb = rows[(2u * j + d) * stride + 4u], sum = rows[(2u * j + d) * stride + 5u];
      if (nb >= q.fl.need && sum / nb < q.fl.threshold) fv |= (uint8_t)(1u << d);
    }
    q.fl.flags[(uint64_t)w * q.fl.n_sites + site] = fv;
  }
}

// Workgroups 0 .. n_windows * tiles - 1: one per (window, tile), the first of
// those that share the tile.  Beyond: q.more per window, the e-th of a window
// taking the e-th share of its shared tiles, if there are that many.  LDS rows
// of eight u64 words: flows, bulk flows, bytes, packets, duration, rate sum,
// min, max (the device-table order).
__global__ __launch_bounds__(kTableThreads, 8) void table_reduce_kernel(const Merge q) {
  extern __shared__ __align__(16) u64 t[];
  __shared__ uint32_t s_sum[kTableThreads / 64], s_all[kTableThreads / 64], s_tile, s_share, s_b[2];
  __shared__ Looked s_look[64];
  const uint32_t lane = threadIdx.x % 64u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64u);
  uint32_t w, tile, share = 0;
  if (blockIdx.x < q.n_windows * q.tiles) {
    w = blockIdx.x / q.tiles;
    tile = blockIdx.x - w * q.tiles;
  } else {
    const uint32_t all = sum_hot(q, s_all);
    if (all == 0u) return;
    const uint32_t x = blockIdx.x - q.n_windows * q.tiles;
    w = x / q.more;
    const uint32_t e = x - w * q.more;
    // the tile whose shares, counted over the tiles, hold share e: every lane
    // sums a run of neighbouring tiles
    const uint32_t per = (q.tiles + kTableThreads - 1u) / kTableThreads, t0 = threadIdx.x * per;
    uint32_t mine = 0;
    for (uint32_t j = t0; j < t0 + per && j < q.tiles; ++j) mine += split_of(q, q.hot[j], all);
    uint32_t incl = mine;
#pragma unroll
    for (uint32_t o = 1; o < 64u; o <<= 1) {
      const uint32_t y = __shfl_up(incl, o, 64);
      if (lane >= o) incl += y;
    }
    if (lane == 63u) s_sum[wave] = incl;
    if (threadIdx.x == 0u) s_share = 0u;
    __syncthreads();
    uint32_t before = incl - mine;
    for (uint32_t v = 0; v < wave; ++v) before += s_sum[v];
    if (e >= before && e < before + mine) {
      for (uint32_t j = t0;; ++j) {
        const uint32_t n = split_of(q, q.hot[j], all);
        if (e < before + n) {
          s_tile = j;
          s_share = e - before + 1u;
          break;
        }
        before += n;
      }
    }
    __syncthreads();
    share = s_share;
    if (share == 0u) return;
    tile = s_tile;
  }
  tile = __builtin_amdgcn_readfirstlane(tile);
  share = __builtin_amdgcn_readfirstlane(share);
  const uint32_t hot = q.more ? q.hot[tile] : 0u;
  const uint32_t tile_rows = 1u << q.tile_bits, r0 = tile << q.tile_bits;
  const uint32_t kind_shift = kEntRowShift + q.tile_bits, window_shift = kind_shift + kEntKindBits;
  const uint32_t nr = q.rows - r0 < tile_rows ? q.rows - r0 : tile_rows;
  u64 *acc = q.acc + ((uint64_t)w * q.rows + r0) * 8u;
  // the window's records, as the classify kernel cuts them: the first window
  // starts at record 0, the last ends at record n
  uint64_t wlo = 0, whi = q.n;
  if (q.woff) {
    if (w > 0) wlo = q.woff[w] < q.n ? q.woff[w] : q.n;
    if (w + 1u < q.n_windows) whi = q.woff[w + 1u] < q.n ? q.woff[w + 1u] : q.n;
  }
  // The nb classify workgroups from bfirst on whose slices may meet it, looked
  // up 64 at a time, a lane for each: slice and entries of the part.  Of up to 64
  // the first wave looks them up for all (16 waves' divisions would bound a call
  // of many small windows); a tile without entries, as most are in a small
  // window, then has nothing to add, only its flags to test.
  uint32_t bfirst = 0, nb = 0, in_l = 0, cap_l = 0;
  uint64_t lo_l = 0, hi_l = 0;
  auto look_up = [&](uint32_t k0, uint32_t step) {
    const uint32_t kl = k0 + lane * step, bl = bfirst + (kl < nb ? kl : 0u);
    lo_l = part_lo(q, bl);
    hi_l = part_lo(q, bl + 1u);
    cap_l = table_range(hi_l - lo_l, q.extra, q.tiles).cap;
    const bool meets = kl < nb && lo_l < whi && hi_l > wlo && lo_l < hi_l;
    in_l = meets ? q.count[(uint64_t)bl * q.tiles + tile] : 0u;
  };
  if (wave == 0u) {
    if (wlo < whi) {
      bfirst = (uint32_t)scaled(wlo, q.grid, q.n);
      bfirst = bfirst ? bfirst - 1u : 0u;
      const uint32_t blast = (uint32_t)scaled(whi - 1u, q.grid, q.n) + 1u;
      nb = (blast < q.grid ? blast : q.grid - 1u) - bfirst + 1u;
    }
    if (nb <= 64u) {
      look_up(0u, 1u);
      s_look[lane] = Looked{lo_l, hi_l, cap_l, in_l};
    }
    if (lane == 0u) {
      s_b[0] = bfirst;
      s_b[1] = nb;
    }
  }
  for (uint32_t r = threadIdx.x; r < tile_rows; r += kTableThreads) {
#pragma unroll
    for (uint32_t f = 0; f < 8u; ++f) t[r * kRowWords + f] = f == 6u ? ~0ull : 0ull;
  }
  __syncthreads();
  bfirst = __builtin_amdgcn_readfirstlane(s_b[0]);
  nb = __builtin_amdgcn_readfirstlane(s_b[1]);
  const bool few = nb <= 64u;
  if (few) {
    const Looked x = s_look[lane];
    lo_l = x.lo;
    hi_l = x.hi;
    cap_l = x.cap;
    in_l = x.in;
    if (__builtin_amdgcn_ballot_w64(in_l != 0u) == 0ull) {
      if (share == 0u && q.fl.flags) flag_rows(q, w, r0, nr, acc, 8u);
      return;
    }
  }
  const uint32_t shares = hot ? 1u + split_of(q, hot, sum_hot(q, s_all)) : 1u;
  // one entry into its row
  auto add = [&](u64 v, u64 y) {
    u64 *o = t + ((uint32_t)(y >> kEntRowShift) & (tile_rows - 1u)) * kRowWords;
    const uint32_t kind = (uint32_t)(y >> kind_shift) & 7u;
    if (kind == kRec) {
      const u64 bytes = y & ((1ull << kEntBytesBits) - 1ull);
      const uint32_t packets = (uint32_t)v, dur = (uint32_t)(v >> 32);
      atomicAdd(&o[0], 1ull);
      atomicAdd(&o[1], bytes);
      atomicAdd(&o[2], (u64)packets);
      atomicAdd(&o[3], (u64)dur);
      if (bytes > q.bulk.bulk_bytes && dur != 0u && bytes >= (u64)q.bulk.min_avg_packet_bytes * packets &&
          packets >= q.bulk.min_packets && dur >= q.bulk.min_duration_ms) {
        const u64 rate = rate_bps(bytes, dur);
        atomicAdd(&o[4], 1ull);
        atomicAdd(&o[5], rate);
        atomicMin(&o[6], rate);
        atomicMax(&o[7], rate);
      }
    } else if (kind == kRowCnt) {  // flows, and bulk flows above them
      atomicAdd(&o[0], v & 0xFFFFFFFFull);
      if (v >> 32) atomicAdd(&o[4], v >> 32);
    } else if (kind == kRowRateMin) {
      atomicMin(&o[6], v);
    } else if (kind == kRowRateMax) {
      atomicMax(&o[7], v);
    } else {  // bytes, packets, duration: words 1..3; rate sum: 5
      atomicAdd(&o[kind == kRowRateSum ? 5u : kind - kRowBytes + 1u], v);
    }
  };
  // A wave of the tile's workgroups for each of the nb, or several where there
  // are fewer of them than waves; four entries per lane in flight.
  constexpr uint32_t U = 4;
  const uint32_t waves = shares * (kTableThreads / 64u), me = share * (kTableThreads / 64u) + wave;
  const uint32_t subs = waves > nb ? waves / nb : 1u, sub = waves > nb ? me / nb : 0u;
  const uint32_t mine0 = sub < subs ? me - sub * nb : nb;  // the wave's first (nb: a wave too many)
  const uint32_t step = few ? 1u : (waves < nb ? waves : nb);
  uint64_t own = ~0ull;
  if (few) {
    own = 0ull;
    for (uint32_t l = mine0; l < nb; l += waves) own |= 1ull << l;
  }
  for (uint32_t k0 = few ? 0u : mine0; k0 < nb; k0 += 64u * step) {
    if (!few) look_up(k0, step);
    for (uint64_t todo = __builtin_amdgcn_ballot_w64(in_l != 0u) & own; todo; todo &= todo - 1u) {
      const uint32_t l = (uint32_t)__builtin_ctzll(todo);
      const uint32_t in = (uint32_t)__builtin_amdgcn_readlane((int)in_l, l), b = bfirst + k0 + l * step;
      const uint64_t lo = readlane64(lo_l, l), hi = readlane64(hi_l, l);
      const char *range = q.entry + kTableRangeBytes * (lo + (uint64_t)b * q.extra);
      const TableEntry *e = (const TableEntry *)range + (uint64_t)tile * (uint32_t)__builtin_amdgcn_readlane((int)cap_l, l);
      // the window's entries (of a short part, all: they are tested below, and a
      // search takes a round trip for every halving)
      uint32_t i0 = 0, end = in & ~kTableMore;
      if (end > U * 64u) {
        if (lo < wlo) i0 = first_of_window(e, end, w, window_shift);
        if (hi > whi) end = i0 + first_of_window(e + i0, end - i0, w + 1u, window_shift);
      }
      // then the tile's chunks, as places after the part's: place i of them
      // all is place i mod chunk of chunk i / chunk
      const uint32_t in_part = end - i0;
      e += i0;
      uint32_t places = in_part, bits = 0;
      const TableChunk *list = nullptr;
      const TableEntry *ce = nullptr;
      if (in & kTableMore) {
        const TableRange rg = table_range(hi - lo, q.extra, q.tiles);
        const uint32_t *first = (const uint32_t *)(range + rg.first) + tile;
        list = (const TableChunk *)(range + rg.list()) + first[0];
        ce = (const TableEntry *)(range + rg.entries());
        bits = rg.bits;
        places += (first[1] - first[0]) << bits;
      }
      for (i0 = sub * U * 64u; i0 < places; i0 += subs * U * 64u) {
        u64x2 x[U];
        uint32_t mine = 0;
#pragma unroll
        for (uint32_t j = 0; j < U; ++j) {
          uint32_t i = i0 + j * 64u + lane;
          const TableEntry *at = e + i;
          bool ok = i < in_part;
          if (!ok && i < places) {
            i -= in_part;
            const u32x4 c = *(const u32x4 *)(list + (i >> bits));  // id, first, count, last
            i &= (1u << bits) - 1u;
            at = ce + ((uint64_t)c.x << bits) + i;
            ok = i < c.z && c.y <= w && w <= c.w;
          }
          if (ok) x[j] = *(const u64x2 *)at;
          mine |= (uint32_t)ok << j;
        }
#pragma unroll
        for (uint32_t j = 0; j < U; ++j)
          if (((mine >> j) & 1u) && (uint32_t)(x[j].y >> window_shift) == w) add(x[j].x, x[j].y);
      }
    }
  }
  __syncthreads();
  // the rows of the device table: word f of row r of window w, one word per
  // lane, consecutive lanes on consecutive words
  if (shares == 1u) {
    for (uint32_t i = threadIdx.x; i < nr * 8u; i += kTableThreads) {
      const uint32_t r = i / 8u, f = i % 8u;
      const u64 c = acc[i], s2 = t[r * kRowWords + f];
      const u64 v = f == 6u ? (s2 < c ? s2 : c) : (f == 7u ? (s2 > c ? s2 : c) : s2 + c);
      if (v != c) acc[i] = v;
      if (q.fl.flags) t[r * kRowWords + f] = v;  // the final row, for the flag test
    }
    if (!q.fl.flags) return;
    __syncthreads();
  } else {
    for (uint32_t i = threadIdx.x; i < nr * 8u; i += kTableThreads) {
      const uint32_t r = i / 8u, f = i % 8u;
      const u64 s2 = t[r * kRowWords + f];
      if (f == 6u) {
        if (s2 != ~0ull) atomicMin(&acc[i], s2);
      } else if (s2 != 0ull) {
        if (f == 7u) atomicMax(&acc[i], s2);
        else atomicAdd(&acc[i], s2);
      }
    }
    if (!q.fl.flags) return;
    // The last of the tile's workgroups has the final rows.  What the workgroups
    // exchange are device-scope atomics alone, so each wave waits for its own to
    // be done and no cache is written back (a fence for every wave took 130 us
    // with 288 workgroups).
    __builtin_amdgcn_s_waitcnt(kWaitVmem);
    __syncthreads();
    if (threadIdx.x == 0u) s_share = atomicAdd(&q.done[(uint64_t)w * q.tiles + tile], 1u);
    __syncthreads();
    if (s_share != shares - 1u) return;
    for (uint32_t i = threadIdx.x; i < nr * 2u; i += kTableThreads) {
      const uint32_t r = i / 2u, f = 4u + i % 2u;
      t[r * kRowWords + f] = __hip_atomic_load(&acc[r * 8u + f], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
  }
  flag_rows(q, w, r0, nr, t, kRowWords);
}

}  // namespace

hipError_t table_prepare(int dev) {
  static std::mutex mu;
  static bool done[64] = {};
  std::lock_guard<std::mutex> g(mu);
  if (dev >= 0 && dev < 64 && done[dev]) return hipSuccess;
  const hipError_t e = hipFuncSetAttribute((const void *)table_reduce_kernel,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)(8u * kRowWords << kTileBitsMax));
  if (e == hipSuccess && dev >= 0 && dev < 64) done[dev] = true;
  return e;
}

bool table_fits(uint32_t n_windows, uint32_t rows) { return (uint64_t)n_windows * ((rows + 255u) / 256u) <= 16384u; }

// The ranges (kTableRangeBytes per record and extra entry), then the counts:
// at most 4 bytes per workgroup and (window, 256 rows), and 8 more per
// (window, 256 rows), with the alignment of the sections included.
uint64_t table_spill_bytes(uint64_t n, uint64_t grid, uint32_t n_windows, uint32_t rows, uint32_t slots) {
  const uint64_t parts = ((uint64_t)n_windows * ((rows + 255u) / 256u) + 63u) & ~63ull;
  return part_layout(n + grid * table_extra(slots), grid, parts, kTableRangeBytes / 2u).end;
}

TableStage table_stage(void *work, uint64_t n, uint64_t grid, uint32_t n_windows, uint32_t tiles, uint32_t slots) {
  char *wb = (char *)work;
  TableStage t{};
  t.entry = wb;
  t.count = (uint32_t *)(wb + kTableRangeBytes * (n + grid * table_extra(slots)));
  t.hot = t.count + grid * tiles;
  t.done = t.hot + tiles;
  t.more = table_more(n, n_windows);
  t.words = t.more ? tiles + n_windows * tiles : 0u;
  return t;
}

int table_merge_launch(void *work, uint64_t n, uint64_t grid, const uint64_t *window_offsets, uint32_t n_windows,
                       uint32_t rows, uint32_t tile_bits, uint32_t slots, const BulkRule &bulk,
                       unsigned long long *acc, const TableFlags &fl, hipStream_t stream) {
  const uint32_t tiles = table_tiles(rows, tile_bits);
  const TableStage ts = table_stage(work, n, grid, n_windows, tiles, slots);
  Merge q{};
  q.entry = ts.entry;
  q.count = ts.count;
  q.hot = ts.hot;
  q.done = ts.done;
  q.woff = n_windows > 1 ? window_offsets : nullptr;
  q.n = n;
  q.extra = table_extra(slots);
  q.grid = (uint32_t)grid;
  q.acc = (u64 *)acc;
  q.rows = rows;
  q.tiles = tiles;
  q.tile_bits = tile_bits;
  q.n_windows = n_windows;
  q.bulk = bulk;
  q.fl = fl;
  q.more = ts.more;
  hipLaunchKernelGGL(table_reduce_kernel, dim3(n_windows * (q.tiles + q.more)), dim3(kTableThreads),
                     8u * kRowWords << tile_bits, stream, q);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    set_last_error(std::string("table merge kernel: ") + hipGetErrorString(e));
    return GNM_E_HIP;
  }
  return GNM_OK;
}

}  // namespace gnm
