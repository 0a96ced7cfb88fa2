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
      const LaunchOrder order = folded_order(heads, nblk, 4, bwd_single_per_cu(64, true));
      const int launched = end_of_launch(heads, nblk, order.head_set, order.fold_end), heaviest_first = end_of_launch(heads, nblk, order.head_set, 0);
      if (launched > heaviest_first) return printf("%d heads of %d blocks: %d intervals, heaviest first %d\n", heads, nblk, launched, heaviest_first), 1;
    }
  return 0;
}

// Launches that count on it have the heaviest items first: in every XCD no item follows a lighter one.
bool heaviest_first(int heads, int items, int head_set) {
  int last[8] = {0};
  for (int b = 0; b < grid_for(heads, items); b++) {
    const int item = work_item(b, items, head_set).item;
    if (item < last[b % 8]) return false;
    last[b % 8] = item;
  }
  return true;
}
int launches_that_count_on_it_are_heaviest_first() {
  for (int heads = 1; heads <= 128; heads++)
    for (int items = 1; heads * items <= 1100; items++) {
      for (int rounds = 2; rounds <= 4; rounds += 2)
        for (int per_cu = 2; per_cu <= 3; per_cu++) {
          const LaunchOrder order = folded_order(heads, items, rounds, per_cu);
          if (order.fold_end != 0 && !heaviest_first(heads, items, order.head_set)) return printf("%d heads of %d items, up to %d rounds\n", heads, items, rounds), 1;
        }
      if (heads * items > 256 && !heaviest_first(heads, items, quad_head_set(heads, items))) return printf("second round of %d heads of %d items\n", heads, items), 1;
    }
  return 0;
}

int main() {
  if (launches_that_count_on_it_are_heaviest_first()) return 1;
  if (one_workgroup_per_cu_is_not_folded()) return 1;
  return 0;
}
