// CPU test of the row kernels' launch plan (plan.h): every size they take, in
// every precision mode, against what the kernels and the workspace assume.
#include "plan.h"

#include <cstdio>
#include <cstdlib>

#define CHECK(c, n)                                                     \
  do {                                                                  \
    if (!(c)) {                                                         \
      std::printf("FAIL n=%d line %d: %s\n", (int)(n), __LINE__, #c);   \
      std::exit(1);                                                     \
    }                                                                   \
  } while (0)

int main() {
  int taken = 0;
  for (int n = 1; n <= 8192; ++n)
    for (int mode = 0; mode <= 2; ++mode) {
      const lddmm::RowPlan r = lddmm::row_plan(n, mode);
      const bool f64 = mode == lddmm::kFP64;
      if (r.m == 0) {
        CHECK(n > (f64 ? 3072 : 5120), n);
        continue;
      }
      ++taken;
      CHECK(r.m >= (f64 ? 2 : 3) && r.m <= (f64 ? 4 : 5), n);        // kernel instances
      CHECK(r.ig >= 1 && r.ig <= 8 && r.jg >= 1, n);
      CHECK(r.ig * r.jg <= (f64 ? 8 : 16), n);                       // waves of a workgroup
      CHECK(r.jg <= (n + 63) / 64, n);                               // no wave without a tile
      CHECK((n + 63) / 64 <= 72 * r.jg, n);                          // FP32 sums of <= 72 terms
      CHECK(r.ig * r.m <= 64, n);                                    // one wave ends the step
      const int rows = r.ig * r.m;
      CHECK(r.groups * rows >= n && (r.groups - 1) * rows < n, n);   // every row once
      CHECK((size_t)r.groups * 8 <= (size_t)n * lddmm::rec_bytes(mode), n);   // H0 partials fit
    }
  CHECK(taken == 2 * 5120 + 3072, taken);
  // the batched kernels' plans, and the room that a server reserves for them
  int most = 0;
  for (int n = 1; n <= 40000; ++n) {
    const lddmm::RowPlan r = lddmm::batch_plan(n);
    const int rows = r.ig * r.m;
    CHECK(r.m == lddmm::kBatchRows && r.ig * r.jg == lddmm::kBatchWaves, n);
    CHECK(r.groups * rows >= n && (r.groups - 1) * rows < n, n);
    CHECK((size_t)r.groups * 8 <= (size_t)n * lddmm::rec_bytes(lddmm::kFP32), n);
    most = r.groups > most ? r.groups : most;
    CHECK(lddmm::batch_groups(n) == most, n);
  }
  std::printf("row plans ok (%d)\n", taken);
  return 0;
}
