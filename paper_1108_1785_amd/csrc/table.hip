// Merge of spilled accumulator rows (§III.B.2, TransRate Kernel: per-site
// statistics; here for registries whose table does not fit LDS).
//
// The classify kernel stages the rows that miss its LDS row cache, and the
// cached rows it flushes at window changes, as 16-byte entries that lie by
// tile of 256 table rows in every workgroup's range (see table.h).
// table_reduce_kernel gives each (window, tile) one workgroup, which owns
// those rows: it sums the entries of its tile and window, from the part of
// every classify workgroup whose slice meets the window, in an LDS table (one
// LDS atomic per field), adds them into its rows of the device table
// (initialised before the classify kernel unless the call accumulates, and
// holding whatever a workgroup added there with device atomics because a part
// had no room) and applies the mean-rate flag test to the sites of its rows.
// Device-scope atomics run at about 23 G/s on MI355X.
// What bounds it: a classify workgroup's cache requests (a read of the trie
// for most records, and 16 bytes stored per entry: the store costs a request
// whether it lands in L2 or beyond, and gathering a wave's entries in LDS
// before storing them changed nothing, 1,289 against 1,296 us).  Entries of 32
// bytes in the order they came, ordered by three partition kernels (counts,
// scan, scatter) that read and wrote all of them twice more, took 1,179 + 131
// + 5 + 447 + 184 us for 10 windows of 10 M records and 20,000 sites; lying by
// tile as they are written they take 1,289 + 144 us (24-byte entries, two
// stores each: 1,335 + 193).  Tiles of 512 or 1,024 rows (fewer, denser parts)
// gain 5 to 10 % there and lose 8 to 25 % on one window, whose merge then has
// too few workgroups.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <string>

#include "gnm_device.h"
#include "partition.h"
#include "rate.h"
#include "registry.h"
#include "table.h"

namespace gnm {

namespace {

constexpr uint32_t kTableThreads = 1024;

struct Merge {
  const char *entry;
  const uint32_t *count;
  const uint64_t *woff;  // NULL: one window
  uint64_t n, extra;
  uint32_t grid;
  u64 *acc;
  uint32_t rows, tiles, n_windows;
  BulkRule bulk;
  TableFlags fl;
};

typedef u64 u64x2 __attribute__((ext_vector_type(2)));

// First of the part's n entries whose window is at least w (windows ascend).
__device__ __forceinline__ uint32_t first_of_window(const TableEntry *e, uint32_t n, uint32_t w) {
  uint32_t lo = 0, len = n;
  while (len) {
    const uint32_t half = len / 2u;
    if ((uint32_t)(e[lo + half].y >> kEntWindowShift) < w) {
      lo += half + 1u;
      len -= half + 1u;
    } else {
      len = half;
    }
  }
  return lo;
}

// One workgroup per (window, tile).  LDS rows of eight u64 words: flows, bulk
// flows, bytes, packets, duration, rate sum, min, max (the device-table order).
__global__ __launch_bounds__(kTableThreads) void table_reduce_kernel(const Merge q) {
  __shared__ u64 t[kTableTileRows][8];
  const uint32_t w = blockIdx.x / q.tiles, tile = blockIdx.x - w * q.tiles;
  const uint32_t r0 = tile * kTableTileRows;
  const uint32_t nr = q.rows - r0 < kTableTileRows ? q.rows - r0 : kTableTileRows;
  for (uint32_t r = threadIdx.x; r < kTableTileRows; r += kTableThreads) {
#pragma unroll
    for (uint32_t f = 0; f < 8u; ++f) t[r][f] = f == 6u ? ~0ull : 0ull;
  }
  __syncthreads();
  // the window's records, as the classify kernel cuts them: the first window
  // starts at record 0, the last ends at record n
  uint64_t wlo = 0, whi = q.n;
  if (q.woff) {
    if (w > 0) wlo = q.woff[w] < q.n ? q.woff[w] : q.n;
    if (w + 1u < q.n_windows) whi = q.woff[w + 1u] < q.n ? q.woff[w + 1u] : q.n;
  }
  // classify workgroups whose slices meet it, a wave for each; four entries per lane in flight
  const uint32_t lane = threadIdx.x % 64u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64u);
  if (wlo < whi) {
    uint32_t b0 = (uint32_t)(wlo * q.grid / q.n);
    b0 = b0 ? b0 - 1u : 0u;
    for (uint32_t b = b0 + wave; b < q.grid; b += kTableThreads / 64u) {
      const uint64_t lo = slice_lo(b, q.n, q.grid), hi = slice_lo(b + 1u, q.n, q.grid);
      if (lo >= whi) break;
      if (hi <= wlo || lo == hi) continue;
      const uint32_t cap = table_part_cap(hi - lo, q.extra, q.tiles);
      const TableEntry *e = (const TableEntry *)(q.entry + kTableRangeBytes * (lo + b * q.extra)) + (uint64_t)tile * cap;
      uint32_t end = q.count[(uint64_t)b * q.tiles + tile];
      uint32_t i0 = 0;
      if (lo < wlo) i0 = first_of_window(e, end, w);
      if (hi > whi) end = i0 + first_of_window(e + i0, end - i0, w + 1u);
      constexpr uint32_t U = 4;
      for (; i0 < end; i0 += U * 64u) {
        u64x2 x[U];
#pragma unroll
        for (uint32_t j = 0; j < U; ++j) {
          const uint32_t i = i0 + j * 64u + lane;
          if (i < end) x[j] = *(const u64x2 *)(e + i);
        }
#pragma unroll
        for (uint32_t j = 0; j < U; ++j) {
          if (i0 + j * 64u + lane >= end) continue;
          const u64 v = x[j].x, y = x[j].y;
          u64 *o = t[(y >> kEntRowShift) % kTableTileRows];
          const uint32_t kind = (uint32_t)(y >> kEntKindShift) & 7u;
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
        }
      }
    }
  }
  __syncthreads();
  // the rows of the device table: word f of row r of window w, one word per
  // lane, consecutive lanes on consecutive words
  u64 *acc = q.acc + ((uint64_t)w * q.rows + r0) * 8u;
  for (uint32_t i = threadIdx.x; i < nr * 8u; i += kTableThreads) {
    const uint32_t r = i / 8u, f = i % 8u;
    const u64 c = acc[i], s2 = t[r][f];
    const u64 v = f == 6u ? (s2 < c ? s2 : c) : (f == 7u ? (s2 > c ? s2 : c) : s2 + c);
    acc[i] = v;
    if (q.fl.flags) t[r][f] = v;  // the final row, for the flag test
  }
  if (!q.fl.flags) return;
  __syncthreads();
  // mean-rate test of the registered sites whose rows lie in this range
  for (uint32_t j = threadIdx.x; 2u * j < nr; j += kTableThreads) {
    const uint32_t site = r0 / 2u + j;
    if (site >= q.fl.n_sites) continue;
    uint8_t fv = 0;
    for (uint32_t d = 0; d < 2u; ++d) {
      const u64 nb = t[2u * j + d][4], sum = t[2u * j + d][5];
      if (nb >= q.fl.need && sum / nb < q.fl.threshold) fv |= (uint8_t)(1u << d);
    }
    q.fl.flags[(uint64_t)w * q.fl.n_sites + site] = fv;
  }
}

}  // namespace

bool table_fits(uint32_t n_windows, uint32_t rows) { return (uint64_t)n_windows * ((rows + 255u) / 256u) <= 16384u; }

// The ranges (kTableRangeBytes per record and extra entry), then the counts:
// at most 4 bytes per workgroup and (window, tile), with the alignment of the
// sections included.
uint64_t table_spill_bytes(uint64_t n, uint64_t grid, uint32_t n_windows, uint32_t rows, uint32_t slots) {
  const uint64_t parts = ((uint64_t)n_windows * ((rows + 255u) / 256u) + 63u) & ~63ull;
  return part_layout(n + grid * table_extra(slots), grid, parts, kTableRangeBytes / 2u).end;
}

TableStage table_stage(void *work, uint64_t n, uint64_t grid, uint32_t rows, uint32_t slots) {
  char *wb = (char *)work;
  return TableStage{wb, (uint32_t *)(wb + kTableRangeBytes * (n + grid * table_extra(slots)))};
}

int table_merge_launch(void *work, uint64_t n, uint64_t grid, const uint64_t *window_offsets, uint32_t n_windows,
                       uint32_t rows, uint32_t slots, const BulkRule &bulk, unsigned long long *acc,
                       const TableFlags &fl, hipStream_t stream) {
  const TableStage ts = table_stage(work, n, grid, rows, slots);
  Merge q{};
  q.entry = ts.entry;
  q.count = ts.count;
  q.woff = n_windows > 1 ? window_offsets : nullptr;
  q.n = n;
  q.extra = table_extra(slots);
  q.grid = (uint32_t)grid;
  q.acc = (u64 *)acc;
  q.rows = rows;
  q.tiles = table_tiles(rows);
  q.n_windows = n_windows;
  q.bulk = bulk;
  q.fl = fl;
  hipLaunchKernelGGL(table_reduce_kernel, dim3(n_windows * q.tiles), dim3(kTableThreads), 0, stream, q);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    set_last_error(std::string("table merge kernel: ") + hipGetErrorString(e));
    return GNM_E_HIP;
  }
  return GNM_OK;
}

}  // namespace gnm
