// Spilled accumulator tables: the interface between the classify launcher
// (kernels.hip) and the kernels that merge the spilled rows (table.hip).
//
// When a registry's table does not fit LDS, a classify workgroup keeps its
// hot rows in an LDS cache.  With a workspace, the rows that miss the cache
// and the cached rows flushed at the end of each window segment are not added
// to the device table with device-scope atomics: each becomes a staged entry.
// A workgroup's range of the workspace is cut into one part per tile of
// kTableTileRows table rows, with an LDS cursor each, so that the entries lie
// by tile (and in window order within a part) as they are written: one
// workgroup per (window, tile) then sums its parts of every classify
// workgroup of the window in LDS and adds them to its rows of the table, and
// writes their flag bytes.  (An append that finds its part full goes to the
// device table with atomics.)
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "gnm.h"

namespace gnm {

constexpr uint32_t kTableTileRows = 256;  // table rows per partition (even: a site's two rows stay together)

// One staged 16-byte entry, one store.  A record that missed the LDS row cache
// is one entry of kind kRec: packets and duration in `x`, bytes in the low
// bits of `y` (whether it is a bulk flow, and its rate, follow from them; a
// record of more bytes than that field holds goes to the device table).  A
// cached row flushed at a window change is one entry for each of its words,
// the word in `x`; the rate words only when it has bulk flows.
struct __attribute__((aligned(16))) TableEntry {
  unsigned long long x, y;
};
constexpr uint32_t kEntBytesBits = 38;  // `y`: bytes of a record, then row within the tile, kind and window
constexpr uint32_t kEntRowShift = 38, kEntKindShift = 46, kEntWindowShift = 49;
constexpr uint32_t kRec = 0u, kRowCnt = 1u, kRowBytes = 2u, kRowPackets = 3u, kRowDur = 4u, kRowRateSum = 5u,
                   kRowRateMin = 6u, kRowRateMax = 7u;
static_assert(kTableTileRows == 1u << (kEntKindShift - kEntRowShift), "row field");  // and table_fits: 14-bit windows

struct TableStage {
  char *entry;      // workgroup b's range: kTableRangeBytes per record and extra entry before it
  uint32_t *count;  // [grid][tiles]: entries in each part
};

// Workspace bytes of a workgroup's range per record of its slice and per
// extra entry: more than twice the one entry that a record can add, so that
// parts of unequal rows have room.
constexpr uint64_t kTableRangeBytes = 64;

// Room in each classify workgroup's range beyond its records, for the cached
// rows of two flushes (a part without room sends its rows to the device table
// with atomics).
inline uint64_t table_extra(uint32_t slots) { return 6ull * slots; }

// Tiles of a table.
inline uint32_t table_tiles(uint32_t rows) { return (rows + kTableTileRows - 1u) / kTableTileRows; }

// Entries in each part of a range over `records` records.
inline __host__ __device__ uint32_t table_part_cap(uint64_t records, uint64_t extra, uint32_t tiles) {
  const uint64_t c = kTableRangeBytes * (records + extra) / (sizeof(TableEntry) * (uint64_t)tiles);
  return c < 0x7FFFFFFFull ? (uint32_t)c : 0x7FFFFFFFu;
}

// Bytes of the spill area of a launch over n records on `grid` workgroups
// with n_windows windows of `rows` rows and `slots` LDS cache slots.
uint64_t table_spill_bytes(uint64_t n, uint64_t grid, uint32_t n_windows, uint32_t rows, uint32_t slots);

TableStage table_stage(void *work, uint64_t n, uint64_t grid, uint32_t rows, uint32_t slots);

// Whether a call of n_windows windows of `rows` rows can spill: at most 16,384
// (window, tile) pairs.
bool table_fits(uint32_t n_windows, uint32_t rows);

// What makes a flow a bulk flow (gnm_params).
struct BulkRule {
  uint64_t bulk_bytes;
  uint32_t min_avg_packet_bytes, min_packets, min_duration_ms;
};

// Flag test fused into the merge (threshold in bits/s; need = max(1, min bulk flows)).
struct TableFlags {
  uint8_t *flags;  // NULL: no flags
  uint64_t threshold, need;
  uint32_t n_sites;
};

// Enqueue the merge after the classify kernel: one workgroup per (window,
// tile) that adds its sums into acc (initialised before the classify kernel,
// or accumulated into) and writes the flags.  window_offsets: as the classify
// kernel got them (NULL: one window).
int table_merge_launch(void *work, uint64_t n, uint64_t grid, const uint64_t *window_offsets, uint32_t n_windows,
                       uint32_t rows, uint32_t slots, const BulkRule &bulk, unsigned long long *acc,
                       const TableFlags &fl, hipStream_t stream);

}  // namespace gnm
