// The rules of dispatch.h on the host: at the shapes where both sides were measured they take the faster one, and what they
// return can be launched.  Prints the first shape that fails and returns 1.
#include <stdio.h>

#include "dispatch.h"

using namespace sage;

// heads, key blocks, d, K-smoothing; long enough for the decoding kernel
const struct { int heads, nblk, d; bool k_smooth, decode; } kDecode[] = {
    {512, 1, 128, true, false}, {4096, 1, 128, true, false}, {512, 1, 64, true, false}, {512, 1, 128, false, true}, {256, 1, 64, true, false},
    {300, 2, 128, true, false}, {400, 2, 128, true, true}, {300, 2, 64, true, true}, {300, 2, 128, false, true}, {128, 4, 128, true, true},
    {64, 8, 128, true, false}, {64, 8, 128, false, true}, {80, 8, 128, true, true}, {64, 8, 64, true, true}, {48, 14, 128, true, true}, {16, 12, 64, true, false},
    {1, 16, 64, true, true}, {1, 16, 128, true, false}, {1, 20, 128, true, true}};
// heads, key blocks, d; workgroups of a head
const struct { int heads, nblk, d, splits; } kSplits[] = {
    {256, 16, 64, 1}, {256, 16, 128, 1}, {256, 8, 64, 1}, {128, 8, 64, 1}, {64, 8, 64, 1}, {192, 12, 128, 1}, {300, 16, 128, 1}, {384, 16, 64, 1},
    {700, 16, 128, 1}, {512, 64, 128, 1}, {180, 12, 64, 1}, {180, 32, 128, 2}, {200, 64, 64, 2}, {240, 12, 128, 1}, {240, 64, 64, 2}, {256, 64, 128, 1}, {64, 128, 128, 8}, {128, 64, 128, 4},
    {64, 32, 64, 4}, {128, 16, 64, 2}, {128, 64, 64, 4}, {150, 64, 128, 3}, {1, 128, 128, 32}, {16, 32, 128, 8}};

// square calls at d = 128: heads, KV blocks, mask; four KV blocks per workgroup measured faster (by 3 % and more on either side)
const struct { int heads, nblk; bool causal, wide; } kBackward[] = {
    {300, 1, true, false}, {520, 1, false, false}, {2048, 1, true, false}, {520, 2, false, false}, {216, 3, true, true}, {280, 3, true, false},
    {480, 3, false, true}, {520, 3, false, false}, {140, 4, false, true}, {184, 4, true, true}, {200, 4, true, true}, {170, 5, false, false},
    {130, 5, true, true}, {110, 5, true, false}, {17, 49, false, true}, {170, 6, false, false}, {130, 6, true, true}, {200, 6, false, true}, {102, 9, false, false}, {102, 9, true, true},
    {86, 10, false, false}, {110, 10, false, true}, {73, 13, false, false}, {65, 13, true, false}, {80, 13, true, true}, {52, 17, true, false},
    {62, 17, true, true}, {40, 18, false, true}, {52, 18, false, false}, {60, 18, false, true}, {43, 21, true, false}, {60, 21, true, true},
    {43, 23, false, false}, {43, 23, true, false}, {40, 25, true, false}, {34, 32, true, false}, {64, 32, true, true}, {64, 32, false, true},
    {30, 33, false, false}, {28, 33, false, true}, {28, 33, true, false}, {20, 50, true, false}, {17, 62, true, false}, {20, 64, true, true},
    {32, 128, true, true}, {64, 128, false, true}};

int splits(int nblk, int per_wave) { return (nblk + 4 * per_wave - 1) / (4 * per_wave); }

int main() {
  for (const auto& c : kDecode)
    if (decode_long_enough(c.heads, c.nblk, c.d, c.k_smooth) != c.decode) return printf("decode_long_enough: %d heads of %d blocks, d %d\n", c.heads, c.nblk, c.d), 1;
  for (const auto& c : kSplits) {
    const int n = splits(c.nblk, decode_blocks_per_wave(c.heads, c.nblk, c.d));
    if (n != c.splits) return printf("decode_blocks_per_wave: %d heads of %d blocks, d %d: %d workgroups\n", c.heads, c.nblk, c.d, n), 1;
  }
  for (const auto& c : kBackward)
    if (bwd_wide_is_faster(c.heads, c.nblk, c.nblk, 0, c.causal) != c.wide) return printf("bwd_wide_is_faster: %d heads of %d blocks, mask %d\n", c.heads, c.nblk, c.causal), 1;
  // four waves per 32 queries: heads, key blocks (as many Q blocks), d, mask
  const struct { int heads, nblk, d; bool causal, quad; } kQuad[] = {{125, 2, 128, true, true}, {125, 2, 64, false, true}, {200, 1, 64, true, false}, {10, 3, 64, true, false},
      {42, 3, 128, true, false}, {32, 4, 64, true, true}, {62, 4, 128, false, true}, {50, 5, 64, true, false}, {25, 5, 128, true, false}, {20, 6, 128, true, true}, {41, 6, 128, true, false},
      {35, 7, 128, false, false}, {35, 7, 64, true, false}, {31, 8, 64, true, false}, {16, 8, 128, true, true}, {27, 9, 64, true, false}, {25, 10, 64, true, true}, {22, 11, 64, true, false},
      {22, 11, 128, true, true}, {20, 12, 64, false, true}, {16, 16, 128, true, true}, {7, 32, 64, true, true}, {28, 9, 128, true, false}, {25, 11, 128, true, false}, {25, 12, 128, true, false},
      {20, 14, 128, true, true}, {18, 16, 128, true, true}, {19, 16, 128, true, false}, {14, 24, 128, true, true}, {12, 32, 128, true, true}, {7, 64, 128, true, true}, {8, 64, 128, true, true},
      {10, 64, 128, true, false}, {5, 128, 128, true, true}, {6, 47, 128, false, false}, {24, 16, 64, true, false}};
  for (const auto& c : kQuad)
    if (fwd_quad_is_faster(c.heads, c.nblk, c.nblk, c.d, c.causal) != c.quad) return printf("fwd_quad_is_faster: %d heads of %d blocks, d %d, mask %d\n", c.heads, c.nblk, c.d, c.causal), 1;
  // psi and the forward in one launch: heads, key blocks, Q blocks, d, the backward's layouts written too
  const struct { int heads, nkblk, nqblk, d; bool share, one; } kShort[] = {{8, 1, 1, 128, true, true}, {4096, 1, 1, 64, false, true}, {384, 1, 32, 64, false, true}, {16, 1, 96, 64, false, false},
      {8, 1, 128, 64, false, true}, {12, 1, 256, 64, false, false}, {256, 1, 128, 128, false, true}, {16, 1, 256, 128, false, false}, {6, 1, 512, 128, false, true}, {64, 1, 64, 128, true, true},
      {32, 1, 128, 128, true, false}, {4, 2, 128, 128, true, false}, {8, 2, 32, 64, false, true}, {16, 2, 64, 128, false, false}, {2048, 2, 2, 128, false, true}, {8, 3, 3, 128, false, false}};
  for (const auto& c : kShort)
    if (fwd_short_is_faster(c.heads, c.nkblk, c.nqblk, c.d, c.share) != c.one) return printf("fwd_short_is_faster: %d heads of %d x %d blocks, d %d\n", c.heads, c.nqblk, c.nkblk, c.d), 1;
  // order of the forward's workgroups: heads, query tiles, Q blocks
  const struct { int heads, tiles, nqblk; bool folded; } kFold[] = {{107, 4, 7, false}, {107, 4, 8, true}, {98, 5, 9, false}, {98, 5, 10, true}, {163, 3, 5, false}, {46, 8, 15, false},
      {64, 8, 15, true}, {80, 5, 9, true}, {245, 2, 3, true}, {51, 10, 19, true}, {36, 14, 28, true}};
  for (const auto& c : kFold)
    if (fwd_is_folded(c.heads, c.tiles, c.nqblk) != c.folded) return printf("fwd_is_folded: %d heads of %d Q blocks\n", c.heads, c.nqblk), 1;
  if (fwd_pair_is_folded(224, 51, 2, 128) || fwd_pair_is_folded(240, 47, 2, 128) || !fwd_pair_is_folded(224, 24, 2, 128) || !fwd_pair_is_folded(224, 62, 2, 64) ||
      !fwd_pair_is_folded(16, 64, 64, 128) || !fwd_pair_is_folded(128, 128, 33, 128))
    return printf("fwd_pair_is_folded\n"), 1;
  // sums of QK-normed keys in the quantiser: row blocks, key blocks
  const struct { int blocks, nkblk; bool fours; } kSums[] = {{1, 1, false}, {4000, 1, false}, {2, 2, true}, {512, 2, true}, {600, 2, false}, {1024, 2, false}, {640, 3, true}, {1280, 3, false},
      {512, 4, true}, {1024, 4, false}, {1024, 8, true}, {2048, 8, true}};
  for (const auto& c : kSums)
    if (normed_rows_by_fours(c.blocks, c.nkblk) != c.fours) return printf("normed_rows_by_fours: %d blocks, %d of a head's keys\n", c.blocks, c.nkblk), 1;
  // Q-smoothing's short table: heads, key blocks, Q blocks, d
  const struct { int heads, nblk, nqblk, d; bool small; } kBias[] = {{1, 1, 1, 128, true}, {16, 16, 16, 128, true}, {32, 8, 8, 128, true}, {18, 16, 16, 128, false},
      {30, 16, 16, 128, false}, {30, 16, 16, 64, false}, {40, 8, 8, 128, false}, {40, 8, 8, 64, true}, {32, 9, 9, 64, false}, {70, 4, 4, 128, false}, {120, 4, 4, 64, true}, {200, 4, 4, 64, false},
      {512, 1, 1, 128, true}, {513, 1, 1, 64, false}, {250, 2, 2, 128, true}, {100, 3, 3, 128, false}, {4, 128, 16, 128, false}, {2, 128, 16, 64, true}, {1, 17, 17, 128, false}};
  for (const auto& c : kBias)
    if (use_bias_short(c.heads, c.nblk, c.nqblk, c.d) != c.small) return printf("use_bias_short: %d heads of %d x %d blocks, d %d\n", c.heads, c.nqblk, c.nblk, c.d), 1;
  // psi(dS) past the caches: heads, key blocks, Q blocks, d, mask; loaded, stored
  const struct { int heads, nblk, nqblk, d; bool causal, load, store; } kTraffic[] = {{36, 28, 28, 128, true, false, false}, {46, 32, 32, 128, true, true, false},
      {64, 32, 32, 128, true, true, false}, {16, 64, 64, 128, false, true, false}, {32, 64, 64, 128, true, true, false}, {64, 64, 64, 128, true, true, true},
      {64, 128, 128, 128, true, true, true}, {1, 1, 1, 64, false, false, false}, {32, 32, 32, 128, false, false, false}, {36, 32, 32, 128, false, true, false},
      {26, 32, 32, 128, false, false, false}, {3, 128, 128, 128, false, false, false}, {12, 64, 64, 64, false, false, false}, {48, 32, 32, 64, false, true, false},
      {20, 64, 64, 64, true, false, false}, {5, 128, 128, 64, true, false, false}, {64, 32, 32, 64, true, true, false}, {120, 16, 16, 128, true, true, false},
      {200, 8, 8, 128, true, false, false}, {40, 128, 16, 128, false, true, false}, {24, 16, 64, 128, false, false, false}, {1, 1040000, 1, 128, false, true, true},
      {700, 4, 4, 128, true, false, false}, {300, 10, 10, 128, true, false, false}, {250, 12, 12, 128, true, false, false}, {400, 12, 12, 128, false, true, false},
      {64, 5, 128, 64, false, false, false}, {74, 3, 132, 64, false, false, false}, {300, 10, 10, 64, false, true, false}, {300, 4, 128, 128, false, true, true}};
  for (const auto& c : kTraffic) {
    const DsTraffic t = ds_traffic(c.heads, c.nblk, c.nqblk, 0, c.d, c.causal);
    if (t.load_past != c.load || t.store_past != c.store) return printf("ds_traffic: %d heads of %d x %d blocks, d %d, mask %d\n", c.heads, c.nqblk, c.nblk, c.d, c.causal), 1;
  }
  // dQ with one Q block per workgroup: heads, key blocks, Q blocks, mask
  const struct { int heads, nblk, nqblk; bool causal, split; } kDq[] = {{1, 1, 1, true, true}, {5000, 3, 1, false, true}, {24, 32, 32, true, true}, {25, 32, 32, true, false},
      {12, 64, 64, true, true}, {13, 64, 64, true, false}, {12, 128, 128, true, true}, {13, 128, 128, true, false}, {16, 32, 32, false, true}, {17, 32, 32, false, false},
      {64, 64, 8, true, true}, {65, 64, 8, true, false},
      // longer walks, and more keys than queries: where the whole step was measured
      {8, 96, 96, true, true}, {16, 64, 64, true, false}, {16, 71, 71, true, false}, {13, 71, 71, true, false}, {16, 82, 82, true, false}, {10, 96, 96, true, false}, {10, 128, 128, true, true},
      {12, 116, 116, true, true}, {10, 141, 141, true, true}, {8, 250, 250, true, false}, {40, 18, 16, true, true}, {40, 24, 16, true, false}, {17, 48, 32, true, true}, {17, 47, 47, true, false}, {11, 99, 66, true, false},
      {31, 32, 16, true, true}, {9, 132, 66, true, false}, {7, 256, 128, true, true}, {26, 48, 16, true, true}, {33, 48, 16, true, false}, {46, 48, 16, true, false}};
  for (const auto& c : kDq)
    if (use_dq_split(c.heads, c.nblk, c.nqblk, c.causal) != c.split) return printf("use_dq_split: %d heads of %d x %d blocks, mask %d\n", c.heads, c.nqblk, c.nblk, c.causal), 1;
  // groups of heads: whole rounds where the walks are even (no mask, or few queries against many keys) and the workgroups have four
  // blocks; else all that fit
  if (bwd_heads_of_group(7, 32, 512, 512, 0, false, true) != 6 || bwd_heads_of_group(9, 16, 128, 128, 0, false, true) != 8 ||
      bwd_heads_of_group(9, 16, 512, 64, 448, true, true) != 8 || bwd_heads_of_group(9, 16, 128, 128, 0, true, true) != 9 ||
      bwd_heads_of_group(9, 16, 128, 128, 0, false, false) != 9 || bwd_heads_of_group(4, 9, 128, 128, 0, false, true) != 4 ||
      bwd_heads_of_group(9, 7, 128, 128, 0, false, true) != 7)
    return printf("bwd_heads_of_group\n"), 1;
  for (int nblk = 1; nblk <= 600; nblk = nblk * 5 / 4 + 1)
    for (int most = 1; most <= 70; most++)
      for (int left = 1; left <= 150; left += 7) {
        const int h = bwd_heads_of_group(most, left, nblk, nblk, 0, false, true);
        if (h < 1 || h > most || h > left || (left > most && h <= most / 2)) return printf("bwd_heads_of_group: %d of %d, %d blocks: %d\n", most, left, nblk, h), 1;
      }
  for (int d = 64; d <= 128; d += 64)
    for (int heads = 1; heads <= 1100; heads++)
      for (int nblk = 1; nblk <= 1200; nblk = nblk < 70 ? nblk + 1 : nblk * 9 / 8) {
        const int per_wave = decode_blocks_per_wave(heads, nblk, d), n = splits(nblk, per_wave);
        // one round of two workgroups per CU, unless a head alone has that many; the partial results (32 rows of O, m, l) fit where K's codes would lie
        const bool fits = n == 1 || (long long)heads * n * 32 * (4 * d + 8) + 256 <= (long long)heads * nblk * 64 * d;
        if (per_wave < 1 || (n > 1 && heads * n > 2 * kCus) || !fits) return printf("%d heads of %d blocks, d %d: %d per wave\n", heads, nblk, d, per_wave), 1;
      }
  return 0;
}
