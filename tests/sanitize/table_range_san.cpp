// Layout of a classify workgroup's range of spilled entries, checked on the
// host: every section lies inside the range and is aligned, and parts and chunks
// together hold every mix of entries over the tiles that the workgroup's records
// and one flush of its row cache can give (all in one tile, evenly over any
// number of neighbouring tiles, one entry too many for every part).
#include <cstdio>
#include <cstdlib>

#include "table.h"

static void check(bool ok, const char *what, uint64_t records, uint64_t extra, uint32_t tiles) {
  if (ok) return;
  std::printf("%s: %llu records, %llu extra, %u tiles\n", what, (unsigned long long)records, (unsigned long long)extra, tiles);
  std::exit(1);
}

// chunks that k entries of a tile take
static uint64_t chunks_for(const gnm::TableRange &r, uint64_t k) {
  return k > r.cap ? (k - r.cap + (1ull << r.bits) - 1u) >> r.bits : 0u;
}

int main() {
  const uint64_t recs[] = {1, 4, 63, 100, 4096, 4099, 39064, 500000, 16777216, 4294967295ull};
  const uint32_t slots[] = {0, 4, 400, 540, 2096, 4096};
  const uint32_t tilec[] = {1, 2, 10, 19, 157, 782, 1024, 2048, 2049};
  for (uint64_t n : recs)
    for (uint32_t s : slots)
      for (uint32_t tiles : tilec) {
        const uint64_t extra = gnm::table_extra(s), room = gnm::kTableRangeBytes * (n + extra);
        const gnm::TableRange r = gnm::table_range(n, extra, tiles);
        const uint64_t C = 1ull << r.bits;
        check(r.cap == (room / (32ull * tiles) < 0x3FFFFFFFull ? room / (32ull * tiles) : 0x3FFFFFFFull), "cap", n, extra, tiles);
        const uint64_t fit = room > r.meta ? (room - r.meta) / (16ull * C + 32u) : 0u;
        check(r.chunks == (fit < gnm::kChunksMax ? fit : gnm::kChunksMax), "number of chunks", n, extra, tiles);
        check(r.bits >= gnm::kChunkBitsMin && r.bits <= gnm::kChunkBitsMax && r.chunks <= gnm::kChunksMax, "fields", n, extra, tiles);
        check(16ull * tiles * r.cap <= r.first && r.first % 16 == 0 && r.first <= room, "parts", n, extra, tiles);
        check(r.chunks == 0 || (r.first + 4ull * (tiles + 1u) <= r.meta && r.meta % 16 == 0), "first", n, extra, tiles);
        check(r.chunks == 0 || r.entries() + 16ull * C * r.chunks <= room, "chunks", n, extra, tiles);
        if (s == 0 || n < 4096 || r.cap < C || n > 16777216) continue;
        // misses, and the words of the rows flushed
        const uint64_t rows = s < n ? s : n, all = n - rows + 7u * rows;
        for (uint32_t m = 1; m <= tiles; ++m)
          check(m * chunks_for(r, (all + m - 1u) / m) <= r.chunks, "even over neighbours", n, extra, tiles);
        const uint64_t full = all / (r.cap + 1ull) < tiles ? all / (r.cap + 1ull) : tiles;
        check(full * chunks_for(r, r.cap + 1ull) <= r.chunks, "one too many each", n, extra, tiles);
      }
  std::printf("table_range_san: ok\n");
  return 0;
}
