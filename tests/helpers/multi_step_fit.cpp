// Prints, for each line "G T cus" of the input, whether a multi-step receding launch fits and
// how many merger blocks and parts it has.  Compiled and run by the CPU test suite.
#include <cstdio>
#include "mppi_types.h"

int main() {
  int G, T, cus;
  while (std::scanf("%d %d %d", &G, &T, &cus) == 3) {
    const bool fits = mppi::multi_step_fits(G, T, cus);
    std::printf("%d %d %d\n", (int)fits, fits ? mppi::merger_blocks(G, T, cus) : 0, mppi::merge_parts(T));
  }
  return 0;
}
