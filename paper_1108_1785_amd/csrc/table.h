// Spilled accumulator tables: the interface between the classify launcher
// (kernels.hip) and the kernels that merge the spilled rows (table.hip).
//
// When a registry's table does not fit LDS, a classify workgroup keeps its
// hot rows in an LDS cache.  With a workspace, the rows that miss the cache
// and the cached rows flushed at the end of each window segment are not added
// to the device table with device-scope atomics: each becomes a staged entry.
// A workgroup's range of the workspace is cut into one part per tile of table
// rows, with an LDS cursor each, so that the entries lie by tile (and in window
// order within a part) as they are written, and, behind the parts, chunks that
// any tile takes when its part is full: one workgroup per (window, tile) then
// sums its parts and chunks of every classify workgroup of the window in LDS
// and adds them to its rows of the table, and writes their flag bytes.  (Only
// when the chunks are used up as well does an entry go to the device table with
// atomics.)
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "gnm.h"

namespace gnm {

// Rows of a tile (even: a site's two rows stay together): 2^8, and more where
// that would be over 1,024 tiles, whose cursors would take the row cache's LDS
// and whose parts would be a few entries each.
constexpr uint32_t kTileBitsMin = 8, kTileBitsMax = 11, kTilesTarget = 1024;

// One staged 16-byte entry, one store.  A record that missed the LDS row cache
// is one entry of kind kRec: packets and duration in `x`, bytes in the low
// bits of `y` (whether it is a bulk flow, and its rate, follow from them; a
// record of more bytes than that field holds goes to the device table).  A
// cached row flushed at a window change is one entry for each of its words,
// the word in `x`; the rate words only when it has bulk flows.
struct __attribute__((aligned(16))) TableEntry {
  unsigned long long x, y;
};
// `y`: bytes of a record, then row within the tile (the tile's bits), kind (3
// bits) and window (15 bits, less those that the row takes beyond 8: table_fits
// leaves tables of wider tiles 16 windows)
constexpr uint32_t kEntBytesBits = 38, kEntRowShift = 38, kEntKindBits = 3;
constexpr uint32_t kRec = 0u, kRowCnt = 1u, kRowBytes = 2u, kRowPackets = 3u, kRowDur = 4u, kRowRateSum = 5u,
                   kRowRateMin = 6u, kRowRateMax = 7u;

struct TableStage {
  char *entry;      // workgroup b's range: kTableRangeBytes per record and extra entry before it
  uint32_t *count;  // [grid][tiles]: entries in each part, and kTableMore when the tile has chunks
  uint32_t *hot;    // [tiles]: entries of the workgroups' fuller parts and of chunks
  uint32_t *done;   // [n_windows][tiles]: merge workgroups that have added their sums of a shared tile
  uint32_t more;    // merge workgroups per window beyond one per tile (0: hot and done are not used)
  uint32_t words;   // of hot and done, which start at 0
};
constexpr uint32_t kTableMore = 0x80000000u;

// Workspace bytes of a workgroup's range per record of its slice and per
// extra entry: four times the one entry that a record can add, half of it in
// parts of one size and half in chunks.
constexpr uint64_t kTableRangeBytes = 64;

// Room in each classify workgroup's range beyond its records, for the cached
// rows of flushes.
inline uint64_t table_extra(uint32_t slots) { return 6ull * slots; }

// Merge workgroups per window beyond one per tile, to share tiles of many
// entries: at most 256 over all windows, and none for the shortest runs (100,000
// records on 1,000 of 1,000,000 sites 252 us a call without, 100 with them; Zipf
// on 20,000 sites, with host statistics, 102 and 77).
inline uint32_t table_more(uint64_t n, uint32_t n_windows) {
  const uint64_t useful = n >> 11;
  return n < (1u << 15) ? 0u : (uint32_t)(useful < 256u ? useful : 256u) / n_windows;
}

// Tiles of a table, and the bits of a tile's rows.
inline uint32_t table_tiles(uint32_t rows, uint32_t bits) { return (rows + (1u << bits) - 1u) >> bits; }
inline uint32_t table_tile_bits(uint32_t rows) {
  uint32_t b = kTileBitsMin;
  while (b < kTileBitsMax && table_tiles(rows, b) > kTilesTarget) ++b;
  return b;
}

// One chunk of a workgroup's range.
struct __attribute__((aligned(16))) TableChunk {
  uint32_t id;     // while staging: the tile it belongs to
  uint32_t first;  // window of its first entry
  uint32_t count;  // entries
  uint32_t last;   // no entry is of a later window
};

// Layout of a range over `records` records: the parts, the first chunk of each
// tile in the list (tiles + 1 words), the chunks' descriptions as they are
// taken, the same listed by tile, the chunks.  A tile that takes chunks has
// filled its part, which is no shorter than a chunk, so that half-filled chunks
// waste no more room than is used.
struct TableRange {
  uint32_t cap;          // entries in a part
  uint32_t bits;         // log2 of the entries in a chunk
  uint32_t chunks;       // chunks there are
  uint64_t first, meta;  // bytes from the range's start
  __host__ __device__ uint64_t list() const { return meta + 16ull * chunks; }
  __host__ __device__ uint64_t entries() const { return meta + 32ull * chunks; }
};
// A tile's chunk cursor: kTableMore, its present chunk, and the entries taken of it.
constexpr uint32_t kChunkBitsMin = 3, kChunkBitsMax = 8;
constexpr uint32_t kUsedBits = 13, kChunksMax = (1u << (31u - kUsedBits)) - 1u;

inline __host__ __device__ TableRange table_range(uint64_t records, uint64_t extra, uint32_t tiles) {
  TableRange r{};
  const uint64_t room = kTableRangeBytes * (records + extra);
  // room / (2 entries * tiles), and the chunks that the rest has room for, in doubles (a 64-bit division takes
  // a wave a microsecond): a quotient is within 2^-13 of the true one, which is no closer below a whole number
  // than 1 / 4,128
  const uint64_t cap = (uint64_t)((double)(kTableRangeBytes / (2u * sizeof(TableEntry)) * (records + extra)) / (double)tiles);
  r.cap = cap < 0x3FFFFFFFull ? (uint32_t)cap : 0x3FFFFFFFu;
  r.bits = kChunkBitsMin;
  while (r.bits < kChunkBitsMax && (2u << r.bits) <= r.cap) ++r.bits;
  r.first = sizeof(TableEntry) * (uint64_t)tiles * r.cap;
  r.meta = r.first + ((4u * ((uint64_t)tiles + 1u) + 15u) & ~15ull);
  const double chunk = (double)((sizeof(TableEntry) << r.bits) + 2u * sizeof(TableChunk));
  const uint64_t chunks = room > r.meta ? (uint64_t)((double)(room - r.meta) / chunk) : 0u;
  r.chunks = chunks < kChunksMax ? (uint32_t)chunks : kChunksMax;
  return r;
}

// Bytes of the spill area of a launch over n records on `grid` workgroups
// with n_windows windows of `rows` rows and `slots` LDS cache slots.
uint64_t table_spill_bytes(uint64_t n, uint64_t grid, uint32_t n_windows, uint32_t rows, uint32_t slots);

TableStage table_stage(void *work, uint64_t n, uint64_t grid, uint32_t n_windows, uint32_t tiles, uint32_t slots);

// Whether a call of n_windows windows of `rows` rows can spill: at most 16,384
// pairs of a window and 256 rows.
bool table_fits(uint32_t n_windows, uint32_t rows);

// Kernel attributes of the merge on device dev (once per device, outside any
// graph capture).
hipError_t table_prepare(int dev);

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
// tile), and more for tiles with many entries, which add their sums into acc
// (initialised before the classify kernel, or accumulated into) and write the
// flags.  window_offsets: as the classify kernel got them (NULL: one window);
// tile_bits: as it had.
int table_merge_launch(void *work, uint64_t n, uint64_t grid, const uint64_t *window_offsets, uint32_t n_windows,
                       uint32_t rows, uint32_t tile_bits, uint32_t slots, const BulkRule &bulk, unsigned long long *acc,
                       const TableFlags &fl, hipStream_t stream);

}  // namespace gnm
