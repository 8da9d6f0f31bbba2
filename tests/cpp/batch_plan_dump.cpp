// Prints the batched row kernels' share of the j tiles for each n given: the waves
// that split them and the tiles of a round, then the pairs of an FP32 sum at most.
#include "plan.h"

#include <algorithm>
#include <cstdio>
#include <cstdlib>

int main(int argc, char** argv) {
  for (int k = 1; k < argc; ++k) {
    const int n = std::atoi(argv[k]);
    const lddmm::RowPlan r = lddmm::batch_plan(n);
    const int tiles = ((n + 63) / 64 + r.jg - 1) / r.jg;   // of a wave
    const int round = std::min(tiles, lddmm::batch_round(false));
    std::printf("%d %d %d %d %d\n", n, r.jg, lddmm::batch_round(false), 4 * round, lddmm::kTile);
  }
  return 0;
}
