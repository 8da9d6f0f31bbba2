// CPU test of which landmarks' state the wave that ends a row workgroup's step
// loads (plan.h, row_state): the workgroup's own, which it alone stores, in every
// plan of the row kernels and of the batched ones; and of the i-groups that the row
// kernels have room for.
#include "plan.h"

#include <algorithm>
#include <cstdio>

static bool own_rows(const lddmm::RowPlan& r, int n) {
  const int rows = r.ig * r.m;
  for (int g = 0; g < r.groups; ++g)
    for (int lane = 0; lane < 64; ++lane) {
      const int i = std::min(lddmm::row_state(g * rows, rows, lane), n - 1);   // the load's clamp
      const int end = std::min(n, (g + 1) * rows);
      if (i < g * rows || i >= end) {
        std::printf("FAIL n=%d group %d lane %d reads %d, owns [%d, %d)\n", n, g, lane, i, g * rows,
                    end);
        return false;
      }
      if (lane < rows && g * rows + lane < n && i != g * rows + lane) {
        std::printf("FAIL n=%d group %d lane %d reads %d\n", n, g, lane, i);
        return false;
      }
    }
  return true;
}

int main() {
  for (int n = 1; n <= 5120; ++n)
    for (int mode = 0; mode <= 2; ++mode) {
      const lddmm::RowPlan r = lddmm::row_plan(n, mode);
      if (r.m > 0 && !own_rows(r, n)) return 1;
      if (r.ig > lddmm::kRowGroups) return 1;   // the kernels' LDS for combined sums
    }
  for (int n : {1, 2, 5, 6, 63, 64, 65, 255, 256, 257, 1000, 4099, 8191, 8192, 8193, 9300, 16383,
                16384, 16385, 20001, 65536})
    if (!own_rows(lddmm::batch_plan(n), n)) return 1;
  std::printf("row states ok\n");
  return 0;
}
