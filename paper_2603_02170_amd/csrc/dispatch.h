// Rules on sizes that choose between forms of a kernel and divide its work: plain host functions, which a test calls as well.
#pragma once

namespace sage {

// CUs of the machine: what a launch has to fill (four SIMDs each).
constexpr int kCus = 256;

// ---- decoding: sage_fwd_decode_kernel -----------------------------------------------------------------
// A query block of at most 32 rows that sees every key takes that kernel, which quantises K and V itself, instead of codes in the
// workspace: with a long cache, or with many heads (its code is long, and with little work few workgroups share the cost of
// fetching it).  Whole calls with one query row, us with codes -> this way.  d = 128: 1 head, 16 key blocks 18.6 -> 19.7, 20 20.6 -> 20.3; 16 heads, 20 23.1
// -> 21.2; 64 of 12 24.6 -> 20.6; 128 of 4 20.4 -> 16.2, 86 of 6 20.7 -> 20.3, 48 of 14 25.1 -> 21.3.  With seven or eight blocks a head's
// one workgroup walks two blocks with each wave: 64 heads of 8 19.7 -> 21.0 (without K-smoothing 16.9 -> 16.1), 80 of 8 22.4 -> 21.7.  d = 64: 16 heads of 12 15.1 -> 16.1,
// 1 of 16 16.1 -> 15.0; 64 of 8 16.0 -> 14.1, 128 of 4 15.2 -> 11.9, 300 of 2 15.1 -> 13.1.
// K-smoothing costs this way a launch for the mean, which the quantiser sums by itself in short heads: with one block a head 512 heads
// of d = 128 13.0 -> 17.3, 4096 87.0 -> 89.1, 512 of d = 64 11.3 -> 13.3 (without K-smoothing 12.2 -> 10.1 at d = 128); with two, d =
// 128, 300 heads 16.8 -> 17.6, 340 17.2 -> 17.7, 384 18.7 -> 17.7.
inline bool decode_long_enough(long long heads, int nblk, int d, bool k_smooth) {
  if (nblk >= (d == 64 ? 16 : 20)) return true;
  const long long blocks = heads * nblk;
  if (k_smooth) {
    if (nblk == 1) return false;
    if (d == 128 && nblk == 2) return blocks >= 768;
    if (d == 128 && (nblk == 7 || nblk == 8)) return blocks >= 640;
  }
  return blocks >= 512;
}

// Key blocks of a wave; a workgroup has four waves, and where a head has several workgroups a second kernel joins their results
// (about 3 us, more with many query rows, whose partial results are FP32 rows).
// Two workgroups fit a CU, so long caches take as many as fill one round of them.  A head keeps one workgroup where that alone is as good.
// (a) Up to eight blocks, two for each wave.  us with the fewest blocks per wave -> with one workgroup, 1 and 32 query rows: d = 64, 128
// heads of 8 16.8 -> 14.8, 20.2 -> 15.1, 64 of 8 14.6 -> 14.1, 16.1 -> 14.3; d = 128, 110 of 5 21.1 -> 20.3, 23.3 -> 20.6, 96 of 8 21.4 -> 21.9, 23.8 -> 22.4.
// (b) Between one and two rounds of one workgroup per CU a second one per head fills no CU better: from 171 heads on if the walks are
// short (180 heads of 12, d = 64, 25.1 -> 19.7; of 32, d = 128, 63.7 one, 59.6 two; 200 of 64, d = 64, 68.6 one, 63.4 two), from 241 on always (240 of 64, d =
// 64, 73.1 one, 70.9 two; 256 of 12, d = 128, 38.4 -> 34.2, of 64, 16 query rows, 148.2 two, 146.6 one, 1 row 144.1 two, 146.3 one).
// At d = 64 one workgroup per CU is enough while its waves have two blocks at most: 64 heads of 32 23.2 -> 20.0, 128 of 16 with 32 rows 25.9 -> 23.8;
// 128 of 64 44.7 -> 43.2 with two per CU.
inline int decode_blocks_per_wave(long long heads, int nblk, int d) {
  auto blocks = [&](long long per_cu) {
    long long n = per_cu * kCus / heads;      // workgroups of a head
    if (n < 1) n = 1;
    return (int)((nblk + 4 * n - 1) / (4 * n));
  };
  const bool between = heads > 170 && (heads > 240 || nblk < (d == 64 ? 48 : 32));
  if (nblk <= 8 || between) return (nblk + 3) / 4;
  return d == 64 && blocks(1) <= 2 ? blocks(1) : blocks(2);
}

}  // namespace sage
