// Every row of dO and every Q block that the staging copies of sage_bwd_single_kernel and sage_bwd_wide_kernel read, over all small
// shapes, the rows that a decoding step reads, the tiles and scales of sage_fwd_quad_kernel and the stages of
// sage_bwd_dq_split_kernel, and the (head, item) of every workgroup, from the index functions the kernels themselves use.  Prints the first access that lies
// outside the tensor, or the first workgroup without a (head, item) of its own, and returns 1.
#include <stdio.h>

#include <algorithm>
#include <vector>

#include "common.h"
#include "bwd_kernel.h"
#include "fwd_kernel.h"

int every_workgroup_has_its_own_work() {
  // sets of the heads of an XCD: four, the largest divisor up to eight, all of a few short ones
  const int sets[][3] = {{4, 64, 4}, {4, 40, 5}, {4, 72, 3}, {16, 152, 19}, {16, 248, 31}, {32, 248, 1}, {4, 272, 2}, {4, 296, 1}, {33, 40, 1}};
  for (const auto& c : sets)
    if (sage::head_set_for(c[0], c[1]) != c[2]) return printf("items %d heads %d: set %d\n", c[0], c[1], sage::head_set_for(c[0], c[1])), 1;
  for (int heads = 1; heads <= 272; heads++)
    for (int items = 1; items <= 68; items++)
      for (int always = 0; always < 2; always++) {
        const int set = sage::head_set_for(items, heads, always != 0), grid = sage::grid_for(heads, items);
        std::vector<char> taken(heads * items, 0);
        for (int b = 0; b < grid; b++) {
          const sage::WorkItem w = sage::work_item(sage::folded(b, sage::fold_end(grid, items, 2 + 2 * always, 2)), items, set);
          const bool inside = w.head >= 0 && w.head < heads && w.item >= 0 && w.item < items;
          if (!inside || taken[w.head * items + w.item]) {
            printf("heads %d items %d set %d: workgroup %d has head %d item %d\n", heads, items, set, b, w.head, w.item);
            return 1;
          }
          taken[w.head * items + w.item] = 1;
        }
        const sage::LaunchOrder order = sage::folded_order(heads, items, 2 + 2 * always, 2);
        std::fill(taken.begin(), taken.end(), 0);
        for (int b = 0; b < grid; b++) {
          const sage::WorkItem w = sage::work_item(sage::folded(b, order.fold_end), items, order.head_set);
          if (w.head < 0 || w.head >= heads || w.item < 0 || w.item >= items || taken[w.head * items + w.item]++) return printf("folded: heads %d items %d: workgroup %d\n", heads, items, b), 1;
        }
        if (grid != heads * items) return printf("heads %d items %d: grid %d\n", heads, items, grid), 1;
      }
  return 0;
}

// The loads of K of sage_fwd_decode_kernel: before the loop the wave's first block, in block j the one after it.
int decoding_reads_every_block_once() {
  for (int nk = 1; nk <= 700; nk++)
    for (int per_wave = 1; per_wave <= 5; per_wave++) {
      const int nblk = (nk + 63) / 64, waves = 4 * ((nblk + 4 * per_wave - 1) / (4 * per_wave));
      std::vector<int> read(nk, 0);
      for (int w = 0; w < waves; w++) {
        const int first = w * per_wave, end = first + per_wave < nblk ? first + per_wave : nblk;
        auto load = [&](int j, bool mine) {
          std::vector<char> rows(nk, 0);
          for (int r = 0; r < 64; r++) {
            const int row = sage::decode_row(64 * j + r, mine, nk);
            if (row < 0 || row >= nk) return false;
            rows[row] = 1;
            if (mine && 64 * j + r < nk && row != 64 * j + r) return false;
          }
          for (int r = 0; r < nk; r++) read[r] += rows[r];
          return true;
        };
        bool fine = load(first, first < end);
        for (int j = first; j < end; j++) fine = fine && load(j + 1, j + 1 < end);
        if (!fine) return printf("decoding: %d keys, %d blocks per wave, wave %d\n", nk, per_wave, w), 1;
      }
      for (int r = 1; r < nk; r++)      // (row 0 stands in for the blocks that no wave has)
        if (read[r] != 1) return printf("decoding: %d keys, %d blocks per wave: row %d read %d times\n", nk, per_wave, r, read[r]), 1;
    }
  return 0;
}

// A workgroup of the forward with four waves per 32 queries: n_tiles of a head's nblk key blocks, two an interval.  Three slots are copied
// before the first interval, slot t + 2 in interval t; interval t forms the logits of pair t + 1 from slot t - 1 and adds pair t - 1 to O from it.
int quad_reads_the_tiles_of_its_pairs() {
  const int tile_bytes = 8192;
  for (int nblk = 1; nblk <= 40; nblk++)
    for (int n_tiles = 1; n_tiles <= nblk; n_tiles++) {
      const int last_off = (nblk - 1) * tile_bytes, pairs = (n_tiles + 1) / 2;
      for (int p = -1; p <= pairs + 2; p++)      // intervals 0 .. pairs
        for (int tile = 0; tile < 2; tile++) {
          const int k = sage::quad_k_offset(p, tile, tile_bytes, last_off), v = sage::quad_v_offset(p, tile, tile_bytes, last_off);
          const int want_k = 2 * (p + 2) + tile, want_v = 2 * p + tile;
          const bool inside = k >= 0 && k <= last_off && k % tile_bytes == 0 && v >= 0 && v <= last_off && v % tile_bytes == 0;
          const bool right = (want_k >= n_tiles || k == want_k * tile_bytes) && (want_v < 0 || want_v >= n_tiles || v == want_v * tile_bytes);
          if (!inside || !right) return printf("four waves: %d of %d tiles, slot %d tile %d: K at %d, V at %d\n", n_tiles, nblk, p, tile, k, v), 1;
        }
      for (int t = 0; t + 1 < pairs; t++) {      // (intervals that form logits)
        const int b = sage::quad_scale_block(t);
        if (b != 2 * (t + 1) || b >= n_tiles || b + 1 > nblk) return printf("four waves: %d of %d tiles, interval %d: scales of block %d\n", n_tiles, nblk, t, b), 1;
      }
    }
  return 0;
}

// dQ with one Q block per workgroup: two stages an interval, the loads of interval m + 3 and the copies of m + 2 in interval m.
int dq_stages_exist() {
  for (int n_j = 1; n_j <= 200; n_j++)
    for (int m = 0; m <= n_j / 2 + 3; m++)
      for (int k = 0; k < 2; k++) {
        const int want = 2 * m + k, j = sage::dq_stage(want, n_j);
        if (j < 0 || j >= n_j || (want < n_j && j != want)) return printf("dQ: %d stages, interval %d: stage %d\n", n_j, m, j), 1;
      }
  return 0;
}

int main() {
  if (quad_reads_the_tiles_of_its_pairs() || dq_stages_exist()) return 1;
  if (every_workgroup_has_its_own_work()) return 1;
  if (decoding_reads_every_block_once()) return 1;
  long long copies = 0;
  for (int causal = 0; causal < 2; causal++)
    for (int nq = 1; nq <= 330; nq++)
      for (int nk = 1; nk <= 330; nk++) {
        if (causal && (nk < nq || (nk - nq) % 64 != 0)) continue;
        const int nqblk = (nq + 63) / 64, nkblk = (nk + 63) / 64, sb = causal ? (nk - nq) / 64 : 0;
        // ahead: tiles copied before the loop, row by row clamped; interval t copies dO of tile t + ahead and the operands of phase B
        // of tile t (one KV block per workgroup: T + 2 intervals, two tiles ahead; four: T + 1 and one)
        for (int blocks = 1; blocks <= 4; blocks += 3)
          for (int j = 0; j < nkblk; j += blocks) {
            const int ahead = blocks == 1 ? 2 : 1;
            const int first = causal ? (j - sb > 0 ? j - sb : 0) : 0;
            const sage::SingleWalk walk(nqblk, first);
            auto bad = [&](const char* what, int t, int row) {
              printf("%s: Nq %d Nk %d causal %d KV block %d (%d per workgroup) interval %d row %d\n", what, nq, nk, causal, j, blocks, t, row);
              return 1;
            };
            if (walk.T < 1 || walk.at(0) != nqblk - 1 || walk.at(walk.T - 1) != first) return bad("walk", 0, 0);
            // (the workgroup's other blocks see no Q block below its first one)
            if (causal && j + blocks - 1 < nkblk && first > (j + blocks - 1 - sb > 0 ? j + blocks - 1 - sb : 0)) return bad("first Q block", 0, 0);
            for (int t = 0; t < ahead; t++)
              for (int r = 0; r < 64; r++, copies++) {
                const int want = 64 * walk.at(t) + r, row = sage::dO_row_clamped(want, nq);
                if (row < 0 || row >= nq || (want < nq && row != want)) return bad("first copies", t, row);
              }
            for (int t = 0; t < walk.T + ahead; t++) {
              if (walk.at(t) < 0 || walk.at(t) >= nqblk || (t < walk.T && walk.at(t) != nqblk - 1 - t)) return bad("phase B", t, 64 * walk.at(t));
              for (int r = 0; r < 64; r++, copies++) {
                const int row = 64 * walk.at(t + ahead) + r * walk.loop_row_step();
                if (row < 0 || row >= nq) return bad("phase A", t, row);
                if (t + ahead < walk.T && row != 64 * (nqblk - 1 - t - ahead) + r) return bad("phase A of a tile that is used", t, row);
              }
            }
          }
      }
  printf("%lld rows\n", copies);
  return 0;
}
