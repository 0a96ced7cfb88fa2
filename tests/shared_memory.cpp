// Outputs in the memory of inputs: which calls the forms of one launch may take.  Prints the first that fails and returns 1.
#include <stdio.h>

#include "dispatch.h"

using namespace sage;

int main() {
  static char m[4096];
  const auto at = [](int first, int bytes) { return Memory{m + first, (size_t)bytes}; };
  const Memory Q = at(0, 256), K = at(256, 512), V = at(768, 512), L = at(2000, 16);
  // O, and whether it lies apart: behind everything, over K, over V, in the place of Q, one row into Q, at the end of V, right behind V
  const struct { Memory O; bool apart; } kFwd[] = {{at(1500, 256), true}, {at(256, 256), false}, {at(1000, 256), false}, {at(0, 256), true}, {at(128, 256), false},
                                                   {at(1279, 256), false}, {at(1280, 256), true}};
  for (const auto& c : kFwd)
    if (fwd_outputs_apart(Q, K, V, c.O, L) != c.apart) return printf("O at %d\n", (int)((const char*)c.O.at - m)), 1;
  for (const Memory& x : {Q, K, V})
    if (fwd_outputs_apart(Q, K, V, at(1500, 256), Memory{x.at, 16})) return printf("LSE at %d\n", (int)((const char*)x.at - m)), 1;
  // K as long as Q: the same memory is another workgroup's all the same
  if (fwd_outputs_apart(Q, at(256, 256), V, at(256, 256), L)) return printf("O in the place of K\n"), 1;

  const Memory in[5] = {Q, K, V, at(1280, 256), at(1536, 256)};
  const struct { Memory dQ, dK, dV; bool apart; } kBwd[] = {
      {at(2100, 256), at(2400, 512), at(3000, 512), true}, {at(0, 256), at(256, 512), at(768, 512), true}, {at(1536, 256), at(2400, 512), at(3000, 512), true},
      {at(256, 256), at(2400, 512), at(3000, 512), false}, {at(2100, 256), at(0, 512), at(3000, 512), false}, {at(2100, 256), at(2400, 512), at(1280, 512), false},
      {at(2100, 256), at(768, 512), at(256, 512), true}, {at(2100, 256), at(384, 512), at(3000, 512), false}, {at(1990, 256), at(2400, 512), at(3000, 512), false}};
  for (const auto& c : kBwd) {
    const Memory out[3] = {c.dQ, c.dK, c.dV};
    if (bwd_outputs_apart(in, L, out) != c.apart) return printf("gradients %d\n", (int)(&c - kBwd)), 1;
  }
  return 0;
}
