// CPU test of the length of the row kernels' FP32 sums: a lane's tiles, times the four
// lanes that are added in FP32, against the bound that the public header states.
#include "plan.h"

#include <cstdio>
#include <initializer_list>

int main() {
  for (int n = 1; n <= 8192; ++n)
    for (int mode : {lddmm::kFP32, lddmm::kFP32Comp}) {
      const lddmm::RowPlan r = lddmm::row_plan(n, mode);
      if (r.m == 0) continue;
      const int tiles = ((n + 63) / 64 + r.jg - 1) / r.jg;
      if (4 * tiles > lddmm::kTile) {
        std::printf("FAIL n=%d: sums of %d pairs\n", n, 4 * tiles);
        return 1;
      }
    }
  std::printf("row pairs ok\n");
  return 0;
}
