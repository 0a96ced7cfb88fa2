// Every row of dO and every Q block that the staging copies of sage_bwd_single_kernel read, over all small shapes, and the
// (head, item) of every workgroup, from the index functions the kernels themselves use.  Prints the first access that lies
// outside the tensor, or the first workgroup without a (head, item) of its own, and returns 1.
#include <stdio.h>

#include <vector>

#include "common.h"
#include "bwd_kernel.h"

int every_workgroup_has_its_own_work() {
  for (int heads = 1; heads <= 272; heads++)
    for (int items = 1; items <= 68; items++)
      for (int always = 0; always < 2; always++) {
        const int set = sage::head_set_for(items, heads, always != 0), grid = sage::grid_for(heads, items);
        std::vector<char> taken(heads * items, 0);
        for (int b = 0; b < grid; b++) {
          const sage::WorkItem w = sage::work_item(b, items, set);
          const bool inside = w.head >= 0 && w.head < heads && w.item >= 0 && w.item < items;
          if (!inside || taken[w.head * items + w.item]) {
            printf("heads %d items %d set %d: workgroup %d has head %d item %d\n", heads, items, set, b, w.head, w.item);
            return 1;
          }
          taken[w.head * items + w.item] = 1;
        }
        if (grid != heads * items) return printf("heads %d items %d: grid %d\n", heads, items, grid), 1;
      }
  return 0;
}

int main() {
  if (every_workgroup_has_its_own_work()) return 1;
  long long copies = 0;
  for (int causal = 0; causal < 2; causal++)
    for (int nq = 1; nq <= 330; nq++)
      for (int nk = 1; nk <= 330; nk++) {
        if (causal && (nk < nq || (nk - nq) % 64 != 0)) continue;
        const int nqblk = (nq + 63) / 64, nkblk = (nk + 63) / 64, sb = causal ? (nk - nq) / 64 : 0;
        for (int j = 0; j < nkblk; j++) {
          const int first = causal ? (j - sb > 0 ? j - sb : 0) : 0;
          const sage::SingleWalk walk(nqblk, first);
          auto bad = [&](const char* what, int t, int row) {
            printf("%s: Nq %d Nk %d causal %d KV block %d interval %d row %d\n", what, nq, nk, causal, j, t, row);
            return 1;
          };
          if (walk.T < 1 || walk.at(0) != nqblk - 1 || walk.at(walk.T - 1) != first) return bad("walk", 0, 0);
          for (int t = 0; t < 2; t++)                   // before the loop: tiles 0 and 1, rows clamped one by one
            for (int r = 0; r < 64; r++, copies++) {
              const int want = 64 * walk.at(t) + r, row = sage::dO_row_clamped(want, nq);
              if (row < 0 || row >= nq || (want < nq && row != want)) return bad("first copies", t, row);
            }
          for (int t = 0; t < walk.T + 2; t++) {        // interval t: phase A of tile t + 2, phase B of tile t
            if (walk.at(t) < 0 || walk.at(t) >= nqblk || (t < walk.T && walk.at(t) != nqblk - 1 - t)) return bad("phase B", t, 64 * walk.at(t));
            for (int r = 0; r < 64; r++, copies++) {
              const int row = 64 * walk.at(t + 2) + r * walk.loop_row_step();
              if (row < 0 || row >= nq) return bad("phase A", t, row);
              if (t + 2 < walk.T && row != 64 * (nqblk - 1 - t - 2) + r) return bad("phase A of a tile that is used", t, row);
            }
          }
        }
      }
  printf("%lld rows\n", copies);
  return 0;
}
