// CPU test of the point flow's cut of the landmarks (plan.h, flow_plan): every
// landmark in one chunk, and no chunk longer than an equal share.
#include "plan.h"

#include <algorithm>
#include <cstdio>

int main() {
  for (int n = 1; n <= 40000; ++n) {
    const lddmm::FlowPlan f = lddmm::flow_plan(n);
    const int chunks = 2 * f.pairs;
    int seen = 0, longest = 0;
    for (int c = 0; c < chunks; ++c) {
      const int a = std::min(n, c * f.clen), b = std::min(n, (c + 1) * f.clen);
      seen += b - a;
      longest = std::max(longest, b - a);
    }
    if (seen != n || longest > (n + chunks - 1) / chunks || f.pairs > 8 ||
        (f.pairs & (f.pairs - 1)) != 0) {
      std::printf("FAIL n=%d: %d chunks of up to %d, %d landmarks\n", n, chunks, longest, seen);
      return 1;
    }
  }
  std::printf("flow plans ok\n");
  return 0;
}
