// The rules of the one-launch forms of short heads at shapes where both sides were timed: they take the faster one.  Prints the first shape
// that fails and returns 1.
#include <stdio.h>

#include "dispatch.h"

using namespace sage;

int main() {
  // heads, queries, keys, d, codes written; one launch.  One key block: Q blocks a power of two and not; two of either; two and more Q blocks
  const struct { int heads, nq, nk, d; bool codes, one; } kFwd[] = {
      {8192, 64, 64, 64, true, true}, {4096, 128, 40, 64, true, true}, {512, 2000, 64, 64, true, true}, {2048, 192, 64, 64, false, true}, {512, 192, 64, 64, true, true},
      {4096, 192, 64, 64, true, false}, {100, 320, 64, 64, true, true}, {131, 384, 64, 64, true, false}, {387, 78, 30, 128, true, false}, {1000, 448, 64, 128, false, false}, {387, 128, 128, 64, true, false}, {15000, 128, 65, 64, false, false}, {512, 320, 64, 64, true, false}, {400, 320, 64, 64, false, true}, {1638, 320, 64, 64, false, false},
      {1820, 526, 64, 64, false, false}, {102, 640, 64, 64, true, false}, {200, 1230, 20, 64, false, false}, {204, 320, 64, 128, true, true}, {1024, 320, 64, 128, true, false},
      {568, 576, 64, 128, true, false}, {744, 704, 64, 128, false, false}, {1555, 576, 64, 128, false, true}, {341, 576, 64, 128, false, true},
      {1024, 65, 65, 64, false, true}, {3000, 65, 65, 64, false, false}, {20000, 65, 65, 64, true, false}, {3000, 128, 128, 64, false, true}, {3000, 128, 128, 64, true, false},
      {8192, 50, 128, 64, true, true}, {256, 128, 128, 128, true, true}, {387, 128, 128, 128, false, false}, {512, 128, 128, 128, false, true}, {3000, 65, 65, 128, false, false},
      {6000, 128, 128, 128, true, true}, {512, 65, 65, 128, true, false}, {1500, 80, 80, 128, true, false}, {24, 1024, 128, 128, false, false}, {16, 1024, 128, 128, true, true},
      {8, 4096, 128, 128, true, false}, {170, 192, 70, 128, true, true}, {32, 1024, 128, 64, true, true}};
  for (const auto& c : kFwd)
    if (fwd_short_is_faster(c.heads, (c.nk + 63) / 64, (c.nq + 63) / 64, c.d, c.codes, c.nq, c.nk) != c.one)
      return printf("fwd_short_is_faster: %d heads of %d x %d, d %d, codes %d\n", c.heads, c.nq, c.nk, c.d, c.codes), 1;
  // heads, queries, keys, d, codes shared; one launch
  const struct { int heads, nq, nk, d; bool share, one; } kBwd[] = {
      {8192, 64, 64, 64, true, true}, {8192, 1, 128, 128, true, true}, {512, 128, 64, 64, true, true}, {1024, 128, 64, 64, true, false}, {2048, 100, 33, 64, false, false},
      {768, 100, 33, 64, false, true}, {8192, 128, 128, 64, true, true}, {2048, 65, 10, 128, true, false}, {512, 65, 10, 128, true, true}, {4096, 128, 64, 128, true, true},
      {4096, 100, 33, 128, false, true}, {2048, 65, 65, 128, true, false}, {8192, 65, 65, 128, false, true}, {4096, 112, 112, 128, true, true}, {2048, 65, 128, 128, true, true},
      {8, 129, 64, 128, true, false}};
  for (const auto& c : kBwd)
    if (bwd_short_is_faster(c.heads, c.nq, c.nk, c.d, c.share) != c.one) return printf("bwd_short_is_faster: %d heads of %d x %d, d %d, share %d\n", c.heads, c.nq, c.nk, c.d, c.share), 1;
  // an XCD for every head in the pre-pass: not where a head has one block of keys and at most two of queries
  if (prepass_rows_shared(2, 1) || prepass_rows_shared(1, 1) || !prepass_rows_shared(3, 1) || !prepass_rows_shared(1, 2)) return printf("prepass_rows_shared\n"), 1;
  return 0;
}
