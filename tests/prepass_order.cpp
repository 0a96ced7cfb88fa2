// The workgroups of a pre-pass launch: every (job, head, block) once, in either layout of the grid and with the last rows first; with an
// XCD for each head, workgroup id % 8 is the head's XCD in every job.  Prints the first launch that fails and returns 1.
#include <stdio.h>

#include <vector>

#include <hip/hip_runtime.h>

#include "common.h"
#include "dispatch.h"

using namespace sage;

int main() {
  for (int heads = 1; heads <= 48; heads++)
    for (int blocks = 1; blocks <= 40; blocks++)
      for (int jobs = 1; jobs <= 4; jobs++)
        for (int mode = 0; mode < 3; mode++) {       // as ids come, own XCD, own XCD with the last rows first
          const bool own = mode > 0;
          if (own && !prepass_own_xcd(heads, blocks)) continue;
          const dim3 g = prepass_grid(blocks, heads, jobs, own);
          std::vector<int> seen((size_t)jobs * heads * blocks, 0);
          if ((size_t)g.x * g.y * g.z != seen.size()) return printf("%d x %d x %d: grid\n", jobs, heads, blocks), 1;
          for (unsigned z = 0; z < g.z; z++)
            for (unsigned y = 0; y < g.y; y++)
              for (unsigned x = 0; x < g.x; x++) {
                PrepassItem i = prepass_item(x, y, z, own, heads);
                if (mode == 2) i = last_rows_first(i, blocks, heads);
                const bool in = i.job >= 0 && i.job < jobs && i.head >= 0 && i.head < heads && i.block >= 0 && i.block < blocks;
                const size_t id = x + g.x * (y + (size_t)g.y * z);
                if (!in || seen[((size_t)i.job * heads + i.head) * blocks + i.block]++ != 0 || (own && (int)(id % 8) != i.head % 8))
                  return printf("%d jobs, %d heads, %d blocks, layout %d: workgroup %zu\n", jobs, heads, blocks, mode, id), 1;
              }
        }
  return 0;
}
