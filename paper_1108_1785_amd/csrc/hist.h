// Rate histograms gathered without device-scope atomics: the interface
// between the classify launcher (kernels.hip) and the histogram kernels
// (hist.hip).
//
// With a workspace that holds them, the classify kernel appends one 32-bit
// key per bulk flow of a registered site to its workgroup's staging range
// (workgroup b owns keys [lo_b, lo_b + count[b]), [lo_b, hi_b) being its
// slice of the records, so the range always has room): the flow's histogram
// row over all windows of the call, window * hist_rows + row, above its
// 14-bit rate bucket.  The partition kernels of partition.h then order the
// keys by ranges of rows, and the reduce kernel counts each range in LDS and
// writes its rows of the histograms.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace gnm {

constexpr uint32_t kHistBucketBits = 14;  // staged key: global row << 14 | bucket

struct HistStage {
  uint32_t *key;
  uint32_t *count;           // [grid]: keys staged by each classify workgroup
  uint32_t *phist;           // [grid][nparts]: each classify workgroup's keys per partition
  unsigned long long *over;  // the overflow-slice counter (cleared by the classify kernel when it counts)
  uint32_t shift;            // a partition holds 2^shift rows
  uint32_t nparts;           // partitions (a multiple of 64)
};

// Whether a call over n records in n_windows windows of hist_rows histogram
// rows can stage its keys (at most 65,536 rows over all windows, fewer than
// 2^32 records).
bool hist_stage_fits(uint64_t n, uint32_t n_windows, uint32_t hist_rows);

// Workspace bytes of the staged histograms of such a call on `grid` classify
// workgroups.
uint64_t hist_work_bytes(uint64_t n, uint64_t grid, uint32_t n_windows, uint32_t hist_rows);

// Staging arrays inside a work area laid out for (n, grid, n_windows, hist_rows).
HistStage hist_stage(void *work, uint64_t n, uint64_t grid, uint32_t n_windows, uint32_t hist_rows);

// Whether such a call counts its histograms straight from the staged keys, in
// one kernel without partitions (and so without partition counts), at most:
constexpr uint32_t kDirectGrid = 2048;            // classify workgroups (their ranges are held in LDS)
constexpr uint64_t kDirectRecords = 100u << 10;   // records
constexpr uint64_t kDirectWork = 1ull << 25;      // records x rows
constexpr uint32_t kDirectAddRows = 2560;         // rows, of a call that accumulates
// Three launches cost more than reading every key once per row, up to the
// lines below (classify call and medians, with the partition kernels and with
// hist_direct_kernel).  Records x rows: 16,384 on 2,000 rows 55.6 and 51.4 us,
// 65,536 on 512 rows 42.0 and 37.8, but 30,000 on 2,000 rows 55.8 and 53.9 and
// 100,000 57.5 and 70.9.  Records: what one row's workgroup may have to count;
// 100,000 flows that are all bulk (classify call alone) take as long either
// way, spread over 64 sites (26.0 and 26.0) or in one row (68.2 and 67.0),
// 131,072 more (26.3 and 28.6, 65.3 and 77.0).
// A call that accumulates writes only the rows that its flows are in: the
// partition kernels pass over empty partitions, a workgroup per row has to read
// the keys first.  2,000 rows (partition kernels, direct) 26.5 and 22.8 us for
// 1,000 records, 32.6 and 29.6 for 16,000; 2,800 rows 33.4 and 33.0, 41.4 and
// 42.1 (11,000); 4,000 rows 37.4 and 38.8, 46.5 and 50.0 (8,000); 64,000 rows
// 214 and 440 (500 records).
inline bool hist_direct(uint64_t n, uint64_t grid, uint32_t n_windows, uint32_t hist_rows, bool accumulate) {
  const uint64_t rows = (uint64_t)n_windows * hist_rows;
  return grid <= kDirectGrid && n <= kDirectRecords && n * rows <= kDirectWork && (!accumulate || rows <= kDirectAddRows);
}

// Kernel attributes of the histogram kernels on device dev (once per device,
// outside any graph capture).
hipError_t hist_prepare(int dev);

// Enqueue the histogram kernels after the classify kernel: partition counts
// (left out when the classify kernel counted its keys per partition itself:
// `counted`), their scan (which also sizes the slices of the most popular
// rows), the scatter into row order, and the reduce into hist (n_windows *
// hist_rows rows of 10,001 counts), which overwrites the rows or, with
// accumulate, adds into them.
int hist_pipeline_launch(void *work, uint64_t n, uint64_t grid, uint32_t n_windows, uint32_t hist_rows,
                         uint32_t *hist, bool accumulate, bool counted, hipStream_t stream);

}  // namespace gnm
