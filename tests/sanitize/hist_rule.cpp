// Which calls count their histograms straight from the staged keys: a line per
// call of the arguments (records, workgroups, windows, rows of a window,
// accumulate), 0 or 1.
#include <cstdio>
#include <cstdlib>

#include "hist.h"

int main(int argc, char **argv) {
  for (int i = 1; i + 4 < argc; i += 5)
    std::printf("%d\n", (int)gnm::hist_direct(std::strtoull(argv[i], nullptr, 10), std::strtoull(argv[i + 1], nullptr, 10),
                                              (uint32_t)std::atoi(argv[i + 2]), (uint32_t)std::atoi(argv[i + 3]),
                                              std::atoi(argv[i + 4]) != 0));
  return 0;
}
