// CPU test of the rule that gives a server its kernels (plan.h, batch_blocks), at
// configurations where both families were timed: none gets the one that is a tenth
// slower when its slots are full.
#include "plan.h"

#include <cstdio>

struct Case { int slots, max_n, mode; bool blocks; };

int main() {
  const int c = lddmm::kFP32Comp, s = lddmm::kFP32, d = lddmm::kFP64;
  const Case cases[] = {
      {1, 2000, c, false},  {4, 15000, c, false}, {2, 15500, c, true},  {1, 16384, c, true},  {2, 16384, c, true},
      {1, 32768, c, true},  {2, 32768, c, true},  {1, 65536, c, true},  {12, 500, c, false},
      {12, 1000, c, false}, {12, 2000, c, false}, {8, 4096, c, false},  {4, 8000, c, false},
      {8, 8000, c, false},  {32, 500, c, true},   {16, 1000, c, true},  {32, 1000, c, true},
      {16, 2000, c, true},  {32, 2000, c, true},  {16, 4096, c, true},  {12, 8000, c, true},
      {32, 8192, c, true},  {1, 16384, s, true},  {8, 8000, s, false},  {32, 500, s, true},
      {1, 65536, d, false}, {2, 32768, d, false}, {4, 16384, d, false}, {16, 4096, d, false},
      {8, 8000, d, false},  {24, 500, d, false},  {24, 1000, d, false}, {32, 1000, d, true},
      {16, 8000, d, true},  {32, 8192, d, true},  {1024, 1 << 20, d, true},
      {1024, 1 << 20, c, true}};
  for (const Case& k : cases)
    if (lddmm::batch_blocks(k.slots, k.max_n, k.mode) != k.blocks) {
      std::printf("FAIL %d slots of %d, mode %d\n", k.slots, k.max_n, k.mode);
      return 1;
    }
  std::printf("families ok\n");
  return 0;
}
