// Order in which the partition scan takes the classify workgroups, driven on
// the host over every launch of up to 700 workgroups: part_source is a
// permutation that takes the workgroups of an XCD (b mod 8) one after the
// other, part_next_source follows it, and a scan wave without a share (which
// starts at `grid`) gets an answer too.
#include <cstdio>
#include <vector>

#include "gnm_device.h"

int main() {
  for (uint32_t grid = 1; grid <= 700; ++grid) {
    std::vector<bool> seen(grid, false);
    uint32_t chain = 0, xcd = 0;
    for (uint32_t i = 0; i < grid; ++i) {
      const uint32_t b = gnm::part_source(i, grid);
      if (b >= grid || seen[b] || b != chain || b % gnm::kXcds < xcd) {
        std::printf("grid %u, place %u: workgroup %u\n", grid, i, b);
        return 1;
      }
      seen[b] = true;
      xcd = b % gnm::kXcds;
      chain = gnm::part_next_source(b, grid);
    }
    (void)gnm::part_source(grid, grid);
  }
  std::printf("part_order_san: ok\n");
  return 0;
}
