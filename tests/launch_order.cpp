// The order in which a launch gives out its workgroups, against a model of the machine: workgroup b goes to XCD b % 8, whose 32 CUs
// take the XCD's workgroups in order, each when it has room.  Prints the first launch that fails and returns 1.
#include <stdio.h>

#include <algorithm>
#include <vector>

#include "common.h"
#include "dispatch.h"

using namespace sage;

// When the last workgroup of a kernel with a CU to itself is done, in intervals: under the mask work item j of a head walks nblk - j Q
// blocks, and every workgroup fills and drains its pipeline (3 intervals).
int end_of_launch(int heads, int nblk, int head_set, int fold) {
  std::vector<int> free_at(8 * 32, 0);
  for (int b = 0; b < grid_for(heads, nblk); b++) {
    const WorkItem w = work_item(folded(b, fold), nblk, head_set);
    auto cu = std::min_element(free_at.begin() + 32 * (b % 8), free_at.begin() + 32 * (b % 8) + 32);
    *cu += nblk - w.item + 3;
  }
  return *std::max_element(free_at.begin(), free_at.end());
}

// Square calls under the mask that sage_bwd_single_kernel takes in up to two rounds of one workgroup per CU (d = 64 with Q-smoothing)
int one_workgroup_per_cu_is_not_folded() {
  for (int nblk = 8; nblk <= 200; nblk++)
    for (int heads = 256 / nblk + 1; heads * nblk <= 512; heads++) {
      const int set = head_set_for(nblk, heads), fold = fold_end(grid_for(heads, nblk), nblk, 4, bwd_single_per_cu(64, true));
      const int launched = end_of_launch(heads, nblk, set, fold), heaviest_first = end_of_launch(heads, nblk, set, 0);
      if (launched > heaviest_first) return printf("%d heads of %d blocks: %d intervals, heaviest first %d\n", heads, nblk, launched, heaviest_first), 1;
    }
  return 0;
}

int main() {
  if (one_workgroup_per_cu_is_not_folded()) return 1;
  return 0;
}
