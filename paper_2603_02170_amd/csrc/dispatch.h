// Rules on sizes that choose between forms of a kernel and divide its work: plain host functions, which a test calls as well.
#pragma once

#include <stddef.h>

namespace sage {

// CUs of the machine: what a launch has to fill (four SIMDs each).
constexpr int kCus = 256;

// Workgroups that fit a CU, of the kernels whose launches are folded (see common.h; a test reads registers and LDS from the build).
inline int fwd_per_cu(int d) { return d == 64 ? 3 : 2; }          // sage_fwd_kernel; sage_fwd_pair_kernel: at least two
constexpr int kMaxSweepPerCu = 2;                                 // sage_bwd_kernel, the sweep for the maxima
inline int bwd_single_per_cu(int d, bool q_smooth) { return d == 64 && !q_smooth ? 2 : 1; }

// Walks of about one length: no mask, or few queries against many keys.
inline bool even_walks(int nblk, int nqblk, bool causal) { return !causal || nblk >= 4 * nqblk; }

// Is the forward with four waves of 32 queries per workgroup folded?  The order takes a head's last query tile for its heaviest.  With an
// odd number of Q blocks half of that tile's waves have no queries: it is the longest and yet light, and in short heads it is a
// large part of all workgroups, which the order then pairs the wrong way.  Whole calls with the mask, us, folded -> not.  d = 128:
// 107 heads of N = 420 32.6 -> 31.3, 100 of 448 30.8 -> 30.2, 86 of 540 34.2 -> 32.8, 98 of 576 37.0 -> 36.2, 163 of 320 33.0 ->
// 32.5, 66 of 704 34.2 -> 33.8, 46 of 960 36.2 -> 35.8, but 57 of 960 40.1 -> 40.8; 34 of 1088 35.6 -> 35.3, 43 of 1216 41.3 ->
// 41.6; d = 64: 113 of 320 18.9 -> 18.4, 143 of 320 21.7 -> 21.8, 92 of 420 23.0 -> 22.6, 86 of 540 26.1 -> 25.6, 71 of 704 27.4 ->
// 26.9, 85 of 704 28.0 -> 28.5, 200 of 192 (two tiles) 17.1 -> 17.2, 245 19.3 -> 19.7.  Heads that divide over the XCDs gain all the
// same, by the items being in order over all of them (80 of 576 31.0 -> 32.7, 64 of 960 39.9 -> 42.4; 48 of 832 33.1 -> 32.7).
inline bool fwd_is_folded(long long heads, int n_qtiles, int nqblk) {
  return nqblk == 2 * n_qtiles || heads % 8 == 0 || n_qtiles < 3 || n_qtiles > 8;
}
// And the one with two waves per 32 queries?  Few queries against many keys have walks of about one length, of which no order is the
// better one, and where the codes of an XCD's heads are many times its L2 a head's workgroups should not be as far apart as that
// order has them.  Whole calls with the mask, us, folded -> not, d = 128: 224 heads of 128 queries against 2560 keys 174.0 -> 170.9,
// 3264 209.6 -> 205.8, 3968 258.8 -> 253.6, 240 against 3008 207.6 -> 201.6, 208 against 3008 179.8 -> 180.0, 224 against 2048 144.0 ->
// 144.0, 1536 103.6 -> 103.9, 512 45.6 -> 46.3; 112 of 256 against 2048 80.8 -> 82.1; d = 64, 224 of 128 against 3968 136.0 -> 136.8.
inline bool fwd_pair_is_folded(long long heads, int nblk, int nqblk, int d) {
  return !even_walks(nblk, nqblk, true) || heads * nblk * 64 * d <= (70ll << 20);
}

// ---- forward of few queries: two waves per 32 queries (sage_fwd_pair_kernel) or four (sage_fwd_quad_kernel) ----
// Four while there is a CU for each workgroup of 64 queries, and at d = 128 for some more where the mask makes the second round
// much the lighter.  An interval takes two key blocks: walks of few blocks gain with an even number of them and lose with an odd
// one, more on fuller machines.  Whole calls, us, two waves -> four.
// d = 128: 2 blocks, 128 workgroups 12.9 -> 12.3, 250 15.9 -> 15.4; 3, 126 14.6 -> 14.8; 4, 128 14.8 -> 14.3, 248 18.7 -> 18.3; 5, 125
// 16.4 -> 16.9, 250 18.5 -> 19.2; 7, 245 20.9 -> 22.2; 6, 8 and 9, 60 and 128 1 to 3 % less, 250 1 to 3 % more; 10, 11 and 12, 60
// to 250 1 to 7 % less; 16, 128 23.7 -> 21.6; 32, 224 36.6 -> 31.5.
// d = 64: 2, 128 10.6 -> 10.5; 3, 126 11.9 -> 12.4; 4, 128 12.6 -> 12.0, 248 14.3 -> 14.5; 5, 250 14.7 -> 15.4; 7, 245 16.7 -> 17.9; 6
// and 8 0 to 5 % more; 10, 1 to 4 % less; 11, 1 % more; 12, 1 to 3 % less; 16, 128 19.7 -> 18.8; 32, 224 29.9 -> 27.5.  One block: 9.0
// -> 9.5.
// More workgroups than CUs: 17 blocks and more, 289 29.2 -> 28.1, 323 29.6 -> 30.0; 24, 345 32.8 -> 31.7; 32, 384 38.5 -> 35.3; 64,
// 448 59.2 -> 50.2, 512 58.3 -> 53.5, 640 (one wave) 74.5 -> 79.5; 128, 640 127 -> 110, 768 126 -> 126; 256, 768 228 -> 221; 12 to
// 16, up to two a block more, 276 26.5 -> 26.4, 280 (14) 28.1 -> 25.6, 288 (16) 29.1 -> 27.2, but 300 (12) 26.9 -> 28.2, 304 (16)
// 29.1 -> 29.7; 11, 275 25.6 -> 26.1; without the mask 47, 282 54.9 -> 64.3; d = 64: 16, 384 21.4 -> 23.4.
inline bool fwd_quad_is_faster(long long heads, int nblk, int nqblk, int d, bool causal) {
  const long long wgs = heads * nqblk;
  if (wgs > kCus) return d == 128 && causal && nblk == nqblk && nblk >= 12 && wgs <= kCus + (nblk < 17 ? 2 : 4) * nblk && wgs <= 3 * kCus;
  if (nblk >= 12 || nblk == 2 || nblk == 4 || nblk == 10) return true;
  return d == 128 && (nblk == 11 || (wgs <= kCus / 2 && (nblk == 6 || nblk == 8 || nblk == 9)));
}

// ---- heads of one or two key blocks: psi and the forward in one launch (sage_fwd_short_kernel; same bits) or in two ----
// One launch, and no codes written and read back where nobody wants them, against every Q block's workgroup quantising all of K and V.
// Whole calls, us, two launches -> one.  One key block, d = 128: 8 heads of N = 64 9.4 -> 7.2, 256 12.6 -> 9.0, 1024 32.3 -> 20.0, 4096 120
// -> 64; 2048 of 1 x 64 49.8 -> 26.9; 8 of 4096 x 64 13.6 -> 11.2, 32 32.8 -> 30.7; d = 64, 8 of 64 8.2 -> 5.8, 4096 63.3 -> 42.1, 16
// of 4096 x 64 14.0 -> 13.0.  Two, d = 128: 8 of N = 128 10.4 -> 9.4, 128 13.4 -> 10.5, 512 34.0 -> 26.9, 2048 121 -> 92; 2048 of 1 x 128
// 63 -> 46; d = 64, 64 of 128 9.7 -> 7.5, 2048 65.6 -> 58.5.  Two and many Q blocks: 8 of 2048 x 128, d = 64, 9.5 -> 7.7, 8 of 4096 x
// 128 15.4 -> 15.0, but 16 of 4096 x 128 21.8 -> 26.4, d = 64 15.2 -> 18.0.  Training steps, whose codes are written all the same: 8 of
// 64 25.7 -> 24.0, 512 52.1 -> 50.0, 8 of 128 28.9 -> 28.5, 256 of 128 49.2 -> 49.5.
// Four key blocks: 8 of 256 12.6 -> 14.9, 128 20.6 -> 29.5, d = 64 64 of 256 12.0 -> 11.4, 128 14.6 -> 21.9; three 12.3 -> 13.8.
// One key block and many Q blocks: 64 heads of 2048 x 64 40.3 -> 30.8, d = 64 28.9 -> 22.0; 384 216 -> 164, 126 -> 104; beyond 32 the Q blocks
// of a head follow each other in the two launches: d = 64, 8 of 8192 x 64 14.3 -> 12.9, but 32 35.2 -> 38.6, 256 255 -> 280, 16 of 6144
// 16.9 -> 17.7, 12 of 16384 26.8 -> 30.3; d = 128, 64 of 4096 60.5 -> 55.2, 256 of 8192 437 -> 426, 6 of 32768 42.4 -> 42.6, but 16 of 16384 53.3 ->
// 55.2, 24 of 32768 154 -> 166; with codes 64 of 4096 x 64 64.0 -> 60.3, 32 of 8192 58.9 -> 60.2, 4 of 8192 x 128 15.8 -> 17.1.
//
// With many heads the two launches are the faster ones again, all the more where the codes are written (`codes`: for a backward, or on a
// workspace of the full size).  Each line lies where both were timed, tensors warm and (in brackets) not seen for 700 MB.
// One key block, d = 64.  Up to 32 Q blocks a head, a power of two of them, one launch always (2048 heads of 128 x 64 52 -> 42, with
// codes 54 -> 44; 512 of 2048 183 -> 141): the two launches read such heads' codes, a power of two apart, at three quarters of the rate
// of others.  Three Q blocks: 1365 heads of 192 42 -> 39 (47 -> 45), with codes 45 -> 44 (51 -> 54), 5461 170 -> 172 (4666: 162 -> 173).
// More: 153 of 320 13.6 -> 10.9, 819 40 -> 39 (45 -> 45), but 1638 68 -> 72, 2000 of 448 (114 -> 144), 1820 of 576 120 -> 142; with
// codes 131 of 384 12.5 -> 13.3, 256 of 320 16.6 -> 18.0, 1638 72 -> 78, (2800 130 -> 168), 102 of 640 14.6 -> 15.3, 1820 of 576 131 ->
// 165.
// d = 128, with codes: just over three workgroups per CU 387 of 78 x 30 19.9 -> 21.1, 131 of 384 19.1 -> 20.6, 67 of 768 18.6 -> 20.1.
// 341 of 576 (53 -> 52), but 568 77 -> 76 (77 -> 82), 744 of 704 (115 -> 127), 1555 of 576 (223 -> 210); with codes 204 of 320 25.1 ->
// 23.3, but 1024 83 -> 90 (92 -> 98), 1170 of 448 (145 -> 149), 568 of 576 77 -> 88 (85 -> 97), 910 (142 -> 156), 236 of 832 (57 -> 60).
// Two key blocks and two Q blocks, d = 64: 1024 heads of 65 33 -> 30, 3000 64 -> 76 (72 -> 83), 20000 with codes 450 -> 605; 3000 of 100
// 76 -> 80 (87 -> 94), of 128 85 -> 81 (96 -> 103), 15000 of 128 x 65 365 -> 374; with codes 387 of 128 17.0 -> 19.0, 1024 39 -> 35,
// 3000 94 -> 105 (104 -> 118).  d = 128: 256 heads, a round of two workgroups per CU, 18.6 -> 15.5, 387 22.6 -> 23.7, 512 34 -> 28; 3000
// of 65 119 -> 124 (126 -> 137), with codes 512 28.8 -> 29.4, 1500 70 -> 79; 1500 of 80 with codes 75 -> 80 (81 -> 88).  More Q blocks,
// d = 128: 24 of 1024 (a CU and a half for each) 14.1 -> 14.4, 12 of 2048 13.6 -> 14.1, 8 of 4096 15.1 -> 15.7; with codes 24 of 1024
// 14.6 -> 16.5, 96 of 256 16.4 -> 17.2, 8 of 4096 15.4 -> 17.0, but 170 of 192 x 70 21.8 -> 19.2.
inline bool fwd_short_is_faster(long long heads, int nkblk, int nqblk, int d, bool codes, int nq = 0, int nk = 0) {
  if (nqblk >= 1 << 20 || (codes && nqblk > 64)) return false;      // (the grid counts threads in 32 bits)
  if (nq == 0) nq = 64 * nqblk;
  if (nk == 0) nk = 64 * nkblk;
  const long long wgs = heads * nqblk;
  const bool power_of_two = (nqblk & (nqblk - 1)) == 0;
  if (nkblk == 1 && d == 64) {
    if (nqblk > 32) return wgs <= (codes ? 3 : 4) * kCus;
    if (power_of_two) return true;
    if (nqblk == 3) return !codes || wgs <= 12 * kCus;
    return wgs <= (codes ? 3 : 8) * kCus;
  }
  if (nkblk == 1) {
    if (nqblk > 128) return wgs <= 12 * kCus;
    if (codes && nqblk > 1 && wgs > 3 * kCus && wgs < 1000) return false;
    if (power_of_two || nqblk == 3) return true;
    if (codes) return wgs <= 10 * kCus;
    return nqblk < 7 || heads % 8 != 0 || wgs <= 16 * kCus || wgs > 40 * kCus;
  }
  if (nkblk != 2) return false;
  if (nqblk == 1) return true;
  if (nqblk == 2 && heads > kCus && (codes ? heads < 500 : d == 128 && heads < 430)) return false;
  if (nqblk == 2 && d == 64) return codes ? heads <= 4 * kCus : heads <= (nq >= 112 ? 4000 : 1300);
  if (nqblk == 2) return heads <= (codes ? kCus : 1300) || nq + nk >= 170;
  if (d == 64) return wgs <= 2 * kCus;
  return wgs <= kCus || (wgs <= 2 * kCus && (codes ? nqblk < 8 && wgs > 448 : nqblk < 16));
}

// ---- outputs that lie in the memory of inputs ----
// In the separate launches of a forward K and V, and Q, are quantised before O and LSE are written, and a backward has read Q, K, O and
// LSE before the gradients are: a caller may have O written over K, say.  The forms of one launch write the rows of one workgroup while
// others still read.  What one workgroup alone reads and writes may be the same memory there: O in the place of Q, row for row, and in
// the backward, of which a workgroup has read a whole head before it writes, a gradient in the place of an input of as many rows.
struct Memory {
  const void* at;
  size_t bytes;
};
inline bool meet(const Memory& a, const Memory& b) {
  const size_t x = (size_t)a.at, y = (size_t)b.at;
  return x < y + b.bytes && y < x + a.bytes;
}
inline bool same(const Memory& a, const Memory& b) { return a.at == b.at && a.bytes == b.bytes; }
inline bool fwd_outputs_apart(const Memory& Q, const Memory& K, const Memory& V, const Memory& O, const Memory& LSE) {
  return !meet(O, K) && !meet(O, V) && (!meet(O, Q) || same(O, Q)) && !meet(LSE, Q) && !meet(LSE, K) && !meet(LSE, V);
}
inline bool bwd_outputs_apart(const Memory (&inputs)[5], const Memory& LSE, const Memory (&gradients)[3]) {
  for (const Memory& g : gradients) {
    if (meet(g, LSE)) return false;
    for (const Memory& x : inputs)
      if (meet(g, x) && !same(g, x)) return false;
  }
  return true;
}

// ---- backward of at most two blocks of queries and of keys: one launch (sage_bwd_short_kernel; same bits) or three ----
// Whole training steps (with the forward in one launch), us, three launches -> one.  d = 128: 8 heads of N = 64 24.1 -> 16.8, 256 31.3 ->
// 23.8, 512 49.7 -> 36.0, 4096 306 -> 218; 8 of N = 128 28.3 -> 24.8, 64 31.3 -> 27.4, 256 49.5 -> 41.1, 512 88.7 -> 78.3, 2048 300 -> 279;
// 8 of 128 x 37 24.7 -> 20.0.  d = 64: 20 of N = 33 18.6 -> 13.4, 256 of 64 22.6 -> 16.6, 1024 57.1 -> 38.4; 8 of 128 22.0 -> 18.5, 512
// 56.6 -> 50.8, 2048 188 -> 176.  (More blocks do not fit the LDS.)
//
// A head whose second block of queries or keys has few rows costs the one launch as much as whole blocks do, and the others' workgroups less:
// with many heads they are the faster ones.  Backward alone, us, three -> one, with the codes shared and (without).  Two Q blocks and one of keys:
// d = 64 (a CU has two workgroups), 512 heads of 128 x 64 24.5 -> 23.5 (31 -> 29), 768 33 -> 34 (42 -> 42), 1024 39 -> 44 (51 -> 55), 2048 68 -> 84 (95 ->
// 108), 8192 of 100 x 33 247 -> 308 (327 -> 381); d = 128, 768 of 65 x 10 40 -> 40, 1400 69 -> 74, 2048 97 -> 104, 2048 of 100 x 33 118 -> 126, but of
// 128 x 64 138 -> 139, 4096 275 -> 260 (without 360 -> 317; 308 -> 288 of 100 x 33).  Two of each, d = 128: 1024 of 65 70 -> 67, 2048 135 -> 144, 8192 492 -> 534
// (669 -> 633), 2048 of 80 143 -> 152, of 96 155 -> 160, 4096 299 -> 299, of 112 327 -> 308; d = 64, 2048 of 65 87 -> 86.
// On tensors not seen for 700 MB, shared: d = 64, 1024 of 128 x 64 44 -> 49, 2400 of 100 x 33 80 -> 101; d = 128, 2400 of 65 x 10 127 -> 135, of 65 172
// -> 183, of 100 x 33 154 -> 157, of 128 x 64 185 -> 175.
inline bool bwd_short_is_faster(long long heads, int nq, int nk, int d, bool share) {
  if (nq > 128 || nk > 128) return false;
  if (nq <= 64) return true;
  if (d == 64) return nk > 64 || heads <= (share ? 2 : 3) * kCus;
  if (!share) return true;
  return nk <= 64 ? nk >= 48 || heads <= 900 : nq + nk >= 170 || heads <= 1200;
}

// ---- launches of the forward's pre-pass, and decoding: does a head have an XCD of its own? (prepass_item; same bits) ----
// With K-smoothing every row of K is read twice and more: by the launch that sums it (or by every workgroup that quantises a block of a
// short head) and by the one that quantises it; the chunk sums are read by every workgroup that quantises a block of the head (eight XCDs
// had fetched them all, one does: 7.3 of 79.8 MB past the L2s with 512 queries against 4096 keys); and the forward reads the codes on the head's XCD.
// What a launch has read or written is still in the L2 of its XCD for the next one, as far as it fits: a plain read of 32 MB by one launch after
// the other takes 2.5 us with every workgroup on the XCD of before and 5.7 on the next one (13 and 5.9 TB/s), a write and a read
// of it 9.3 and 24.4; of 48 MB 7.9 either way, but 4.5 with the order reversed every time.  (Profiler runs that count traffic empty the L2s
// before every launch, and show none of this but the chunk sums.)  Whole calls, us, ids as they come -> own XCD, the same tensors every time: forward, 8 heads of N = 1000 22.1 -> 20.3, 8 of 512 17.8 -> 16.3, 64 of 256 16.2 -> 15.5, 128 of 640 49.0 -> 47.3, 200
// of 300 40.3 -> 38.9, 32 of 512 against 4096 keys 60.6 -> 57.0; d = 64, 16 of 512 15.2 -> 14.3, 8 of 2000 25.8 -> 25.2; decoding, 64
// heads of 8192 keys 78.6 -> 76.1; steps, 16 of 512 47.4 -> 45.7, 64 of 2048 and more the same.
// One block a head has nothing to share (8 of 64 9.33 -> 9.38).  Without gain, or with a loss: QK-norm (its sums wait for their
// chains; blocks of 128, 32 of 2048 235.4 -> 238.1), Q-smoothing (the bias kernel reads K in the order of ids, 16 of 1024 31.2 -> 31.9),
// numerics blocks of 128 (32 of 2048 58.7 -> 60.0).  On tensors not seen for 700 MB: 8 of N = 1000 24.1 -> 22.7, 64 of 256 18.7 -> 16.9, 32 of 512 x
// 4096 67.0 -> 62.3, 8 of 8192 x 512 39.9 -> 34.0, d = 64 26.8 -> 23.0; steps, 64 of 2048 343 -> 339.  It does not gain everywhere that it is
// taken: d = 64, 256 heads of 2560 x 313 1.03 times as long, 632 of 2847 x 297 1.04.  (65535: the grid's y and z.)
inline bool prepass_own_xcd(int heads, long long blocks) { return heads % 8 == 0 && blocks > 1 && blocks <= 65535; }
// One block of K and one or two of the others are no more: backwards that quantise Q and K themselves, d = 64, ids as they come -> own XCD,
// 1000 heads of 128 x 64 49.1 -> 50.3, 2000 90.6 -> 93.8; three blocks and more 1000 of 512 x 64 with 7 % less.
inline bool prepass_rows_shared(int nqblk, int nkblk) { return nkblk > 1 || nqblk > 2; }
// dO alone, in a backward that shares psi(Q) and psi(K): the forward has left O, and the backward finds the codes, in the L2 of the head's
// XCD, while the 5 bytes an element of all heads are little more than the L2s hold (32 MB).  Steps, us, ids as they come -> own XCD: 8
// heads of N = 128 29.2 -> 28.8, 128 of 256 55.7 -> 54.6, 32 of 1024 81.5 -> 80.6, 64 of 1024 134.4 -> 132.7, 32 of 2048 183.1 ->
// 182.3; d = 64, 64 of 1024 90.8 -> 90.0; but this launch of 64 of 2048 17.2 -> 18.3.  Backwards alone, on tensors not seen for 700 MB: 128 heads
// of N = 256 36.1 -> 35.7, d = 64 25.4 -> 24.9, 64 of 1024 95.1 -> 94.1, 65.5 -> 64.9.
inline bool dO_own_xcd(long long elements) { return elements <= (8 << 20); }

// ---- quantiser that sums QK-normed keys by itself: four rows at a time, or one at a time with fewer registers ----
// `blocks` = row blocks of 64 of the longer of Q and K over all heads.  Every workgroup of the launch has the registers of those that
// sum, so with many blocks the occupancy counts for more than the chain of a short sum.  Whole forward calls, us, four rows at a time
// -> one, heads of queries x keys.  d = 128: 16 of 1024 x 128 (256 blocks) 15.6 -> 17.0, 32 22.9 -> 22.7, 64 38.1 -> 35.2, 128 of
// 2048 x 128 (4096) 128 -> 113; 300 of 90 (600) 27.4 -> 26.5; 64 of 640 x 192 (640) 26.3 -> 29.8, 128 41.4 -> 41.2; 32 of 1024 x 256
// (512) 27.6 -> 31.2, 64 45.6 -> 43.5, 64 of 2048 x 256 (2048) 83.2 -> 78.4; 16 of 4096 x 512 (1024) 47 -> 62.  d = 64: 32 of 1024 x
// 128 (512) 15.3 -> 15.6, 64 23.7 -> 22.6; 500 of 128 (1000) 25.9 -> 25.3; 64 of 640 x 192 18.2 -> 18.5, 128 24.2 -> 23.0; 32 of
// 1024 x 256 18.0 -> 19.4, 64 27.6 -> 26.8; 32 of 4096 x 512 (2048) 49 -> 55.
inline bool normed_rows_by_fours(long long blocks, int nkblk) {
  return nkblk > 4 || (nkblk > 1 && blocks < (nkblk == 2 ? 600 : 1024));
}

// ---- Q-smoothing's bias table for at most 16 Q blocks: qsmooth_bias_short_kernel or qsmooth_bias_kernel (same bits) ----
// Workgroups (one per key block and head) with a CU to themselves are bound by latency, and the short kernel has no LDS and no
// barrier; where they share one, its narrow loads, of Q's means for every 16 keys again, cost more than that.  Whole forward
// calls that differ in this kernel only, us, qsmooth_bias_kernel -> the short one, by workgroups (heads of N):
// d = 128: 1 (1 of 64) 14.2 -> 13.4, 40 (40 of 41) 14.6 -> 13.7, 64 (8 of 512) 23.2 -> 22.6, 128 (8 of 1000) 28.9 -> 29.0, 256 (16 of
// 1024) 33.3 -> 33.0, (32 of 512) 28.0 -> 27.4, (2 of 1024 against 8192 keys) 73.9 -> 74.0; one Q block: 300 22.8 -> 22.7, 512 26.3
// -> 25.8; two: 300 26.0 -> 26.1, 500 29.0 -> 28.8; three: 300 26.4 -> 26.7; four: 280 27.4 -> 27.8; eight: 320 31.4 -> 32.4; 16:
// 288 36.4 -> 38.7, 480 40.2 -> 42.1, the step 92.4 -> 94.2.
// d = 64: 6 (2 of 130) 14.0 -> 13.2, 208 (13 of 1008) 27.4 -> 26.9, 256 (16 of 1024) 25.4 -> 25.0; one Q block: 500 18.3 -> 17.9, four: 280
// 21.0 -> 20.9, 480 21.5 -> 21.2; eight: 320 23.12 -> 23.10, 384 24.2 -> 24.1; nine: 288 23.2 -> 23.4; 12: 264 26.9 -> 27.3; 16: 288
// 29.7 -> 30.3, 480 33.3 -> 34.1.
// From two workgroups per CU on (d = 128, 800 of four Q blocks 43.2 -> 44.2; d = 64, 748 of seven 31.0 -> 32.0) and from 17 Q blocks on,
// where the larger products have rows for all their lanes, the other kernel.
inline bool use_bias_short(long long heads, int nblk, int nqblk, int d) {
  const long long wgs = heads * nblk;
  return nqblk <= 16 && wgs <= (nqblk <= (d == 64 ? 8 : 2) ? 2 * kCus : kCus);
}

// ---- decoding: sage_fwd_decode_kernel -----------------------------------------------------------------
// A query block of at most 32 rows that sees every key takes that kernel, which quantises K and V itself, instead of codes in the
// workspace: with a long cache, or with many heads (its code is long, and with little work few workgroups share the cost of
// fetching it).  Whole calls with one query row, us with codes -> this way.  d = 128: 1 head, 16 key blocks 18.6 -> 19.7, 20 20.6 ->
// 20.3; 16 heads, 20 23.1 -> 21.2; 64 of 12 24.6 -> 20.6; 128 of 4 20.4 -> 16.2, 86 of 6 20.7 -> 20.3, 48 of 14 25.1 -> 21.3.  With
// seven or eight blocks a head's one workgroup walks two blocks with each wave: 64 heads of 8 19.7 -> 21.0 (without K-smoothing 16.9
// -> 16.1), 80 of 8 22.4 -> 21.7.  d = 64: 16 heads of 12 15.1 -> 16.1, 1 of 16 16.1 -> 15.0; 64 of 8 16.0 -> 14.1, 128 of 4 15.2 ->
// 11.9, 300 of 2 15.1 -> 13.1. K-smoothing costs this way a launch for the mean, which the quantiser sums by itself in short heads:
// with one block a head 512 heads of d = 128 13.0 -> 17.3, 4096 87.0 -> 89.1, 512 of d = 64 11.3 -> 13.3 (without K-smoothing 12.2
// -> 10.1 at d = 128); with two, d = 128, 300 heads 16.8 -> 17.6, 340 17.2 -> 17.7, 384 18.7 -> 17.7.
// (Heads of one or two key blocks have a form of one launch now, which is asked first and takes every such call: what stands here of them
// compares the two that it replaced, and decides nothing.)
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

// A head's workgroups on one XCD (prepass_item), by the elements of K: while K fits the L2s (32 MB in all) the second read of it comes from
// there.  Beyond, an L2 that has passed all of its share has the start of it no longer, and what is left is the chunk sums' one fetch; in
// between calls lost by it, by up to 9 %, for no cause that has been found (the keys of a head count too: 33 MB at d = 64 gained with
// 32 heads and lost with 64), and the ids stay as they come there.  Whole calls with one query row, the same tensors every time, us, ids as they come -> own XCD, MB of K: d = 128: 4 (8 heads of 2048 keys) 18.7 -> 17.5, 17 (8 of 8192) 23.2 ->
// 21.9, 25 (24 of 4096) 26.7 -> 26.2, 33 (16 of 8192) 29.6 -> 29.9, 33 (64 of 2048) 28.3 -> 28.5, 50 (48 of 4096) 39.2 -> 39.4, 67 (64 of
// 4096) 44.6 -> 45.3, 67 (128 of 2048) 45.7 -> 47.8, 100 (96 of 4096) 65.2 -> 64.1, 134 (64 of 8192) 78.4 -> 76.2; d = 64: 8 (32 of 2048) 16.8
// -> 16.0, 17 (32 of 4096) 20.2 -> 19.6, 25 (24 of 8192) 26.7 -> 26.0, 33 (64 of 4096) 29.3 -> 30.3, 33 (32 of 8192) 27.9 -> 26.8, 50
// (96 of 4096) 40.0 -> 41.7, 67 (128 of 4096) 44.6 -> 48.5, 100 (96 of 8192) 63.0 -> 62.5, 134 (128 of 8192) 78.5 -> 77.4.  Larger, and past the
// memory-side cache (256 MB): d = 128, 268 (64 of 16384) 142 -> 143, (32 of 32768) 145 -> 143, (256 of 4096) 145 -> 146, 537 (64 of 32768) 295 -> 288, (1024
// of 2048) 287 -> 288.  On tensors not seen for 700 MB: d = 128, 17 (8 of 8192) 24.5 -> 24.1, 134 (64 of 8192) 82.8 -> 81.4, 268 (64 of 16384) 154.7 ->
// 154.2, 537 (64 of 32768) 309 -> 303, (256 of 8192) 301 -> 302.
inline bool decode_own_xcd(long long elements) { return elements <= (14ll << 20) || elements >= (48ll << 20); }

// Key blocks of a wave; a workgroup has four waves, and where a head has several workgroups a second kernel joins their results
// (about 3 us, more with many query rows, whose partial results are FP32 rows).
// Two workgroups fit a CU, so long caches take as many as fill one round of them.  A head keeps one workgroup where that alone is as good.
// (a) Up to eight blocks, two for each wave.  us with the fewest blocks per wave -> with one workgroup, 1 and 32 query rows: d = 64, 128
// heads of 8 16.8 -> 14.8, 20.2 -> 15.1, 64 of 8 14.6 -> 14.1, 16.1 -> 14.3; d = 128, 110 of 5 21.1 -> 20.3, 23.3 -> 20.6, 96 of 8
// 21.4 -> 21.9, 23.8 -> 22.4. (b) Between one and two rounds of one workgroup per CU a second one per head fills no CU better: from
// 171 heads on if the walks are short (180 heads of 12, d = 64, 25.1 -> 19.7; of 32, d = 128, 63.7 one, 59.6 two; 200 of 64, d = 64,
// 68.6 one, 63.4 two), from 241 on always (240 of 64, d = 64, 73.1 one, 70.9 two; 256 of 12, d = 128, 38.4 -> 34.2, of 64, 16 query
// rows, 148.2 two, 146.6 one, 1 row 144.1 two, 146.3 one). At d = 64 one workgroup per CU is enough while its waves have two blocks
// at most: 64 heads of 32 23.2 -> 20.0, 128 of 16 with 32 rows 25.9 -> 23.8; 128 of 64 44.7 -> 43.2 with two per CU.
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

// ---- backward, d = 128: two KV blocks per workgroup (sage_bwd_kernel) or four (sage_bwd_wide_kernel) ----

// CUs that take workgroups from a queue, one at a time each: when the last one is done, in the unit of the workgroups' times.
class Queue {
 public:
  // `count` workgroups of `time` each, behind those already queued
  void add(long long count, double time) {
    total_ += count * time;
    while (count > 0) {
      const Level first = level_[0];              // the CUs that are free first
      const long long n = count < first.cus ? count : first.cus;
      if (n == first.cus) {
        for (int k = 1; k < levels_; k++) level_[k - 1] = level_[k];
        levels_--;
      } else {
        level_[0].cus -= n;
      }
      put(first.time + time, n);
      count -= n;
    }
  }
  // (a machine that runs dry speeds up: part of the estimate is the mean over the CUs)
  double end() const { return 0.85 * level_[levels_ - 1].time + 0.15 * total_ / kCus; }

 private:
  struct Level {
    double time;
    long long cus;
  };
  void put(double time, long long cus) {
    int k = levels_;
    while (k > 0 && level_[k - 1].time > time) k--;
    if (k > 0 && level_[k - 1].time == time) {
      level_[k - 1].cus += cus;
      return;
    }
    for (int m = levels_; m > k; m--) level_[m] = level_[m - 1];
    level_[k] = {time, cus};
    levels_++;
  }
  Level level_[kCus + 1] = {{0.0, kCus}};         // in order; every level has a CU
  int levels_ = 1;
  double total_ = 0.0;
};

// Both kernels run one workgroup per CU, heaviest first.  In units of an interval with two KV blocks, a workgroup with two takes its
// walk and 5 for filling and draining, one with four 1.65 times its walk and 3; with at most half of its blocks there it takes 0.8 of
// that (numbers fitted to 576 shapes: heads of 1 to 72 KV blocks, 400 to 3000 blocks in all, with the mask and without; the
// choice then costs 0.1 % on average against the better side of each, at most 7 %).
struct BwdEstimate {
  double two, four;
};
inline BwdEstimate bwd_estimate(long long heads, int nblk, int nqblk, int shift_blocks, bool causal) {
  Queue two, four;
  if (even_walks(nblk, nqblk, causal)) {
    two.add(heads * (nblk / 2), nqblk + 5);
    if (nblk % 2 != 0) two.add(heads, 0.8 * (nqblk + 5));
    const int rest = nblk % 4;
    four.add(heads * (nblk / 4 + (rest == 3)), 1.65 * (nqblk + 3));
    if (rest == 1 || rest == 2) four.add(heads, 0.8 * 1.65 * (nqblk + 3));
  } else {
    auto walk = [&](int j) { return nqblk - (j > shift_blocks ? j - shift_blocks : 0); };
    for (int j = 0; j < nblk; j += 2) two.add(heads, (nblk - j > 1 ? 1.0 : 0.8) * (walk(j) + 5));
    for (int j = 0; j < nblk; j += 4) four.add(heads, (nblk - j > 2 ? 1.65 : 0.8 * 1.65) * (walk(j) + 3));
  }
  return {two.end(), four.end()};
}

// Four KV blocks per workgroup?  Whole backward calls, us, two -> four.  Without
// the mask: 32 heads of N = 1024 65.6 two (one round), 34 104 -> 85; 102 of 576 82.8 -> 92.5 (two rounds either way), 110 100.4 ->
// 97.2; 30 of 2112 206 -> 241, 16 of 4160 502 -> 470; 520 of 64 38.1 -> 45.4, 140 of 256 51.5 -> 43.1, 170 of 320 62.5 -> 68.0.
// With it: 34 of 2048 139.7 -> 143.8, 36 148.6 -> 145.6; 43 of 1344 92.3 -> 101.6, 60 121 -> 108; 20 of 3200 177 -> 202, 20 of 4096
// 284 -> 270; 520 of 64 40.4 -> 45.4, 216 of 192 45.0 -> 37.0.  Numerics blocks of 128 and Q-smoothing have the same lines (34 of
// 2048, blocks of 64 x 128 140 -> 144, 128 x 64 179 -> 183, 128 x 128 180 -> 186; 36 151 -> 145, 189 -> 185, 191 -> 188).
inline bool bwd_wide_is_faster(long long heads, int nblk, int nqblk, int shift_blocks, bool causal) {
  // (one and two blocks leave half of the workgroup idle; one round of workgroups with two blocks each is never longer, nor a little
  // more than one of short walks with the mask: 110 heads of 320 40.7 -> 42.8, 97 of 384 48.0 -> 46.5)
  if (nblk <= 2 || heads * nblk <= (causal && nblk > 4 ? 9 * kCus / 4 : 2 * kCus)) return false;
  // three: 272 heads 49.3 -> 55.6 with the mask, 300 without 59.7 -> 60.6, 480 79.6 -> 71.6, 520 88.2 -> 92.7, 573 99.1 -> 95.2
  if (nblk == 3) return heads <= kCus || (heads - 1) % kCus >= 48;
  const long long wgs = heads * ((nblk + 3) / 4);
  if (wgs >= 4 * kCus) return true;
  const bool even = even_walks(nblk, nqblk, causal);
  // (long walks of all lengths: the longest one decides; 272 workgroups of N = 4096 188 -> 207, 304 270 -> 270, 320 225 -> 214)
  if (!even && nblk > 64) return wgs > kCus * 6 / 5;
  const BwdEstimate t = bwd_estimate(heads, nblk, nqblk, shift_blocks, causal);
  // (where both are near, the estimate is 2 % too good for two blocks with the mask, 35 heads of 2048 149 -> 146, 20 of 4096 284 ->
  // 270, and 3 % for long walks without, 24 of 3776 528 -> 508, 16 of 4160 502 -> 470)
  return t.four < (!even ? 1.02 : nblk > 48 ? 1.03 : 1.0) * t.two;
}

// Heads of the next group of a backward whose psi(dS) does not fit the scratch at once: `most` do, `left` are left.  Where all
// workgroups run for about the same time a group takes whole rounds of them, so the size is the one with the shortest estimate in all,
// the largest of those (32 heads of N = 32768 without the mask: 7 heads fill three and a half rounds of workgroups with four KV
// blocks and take 7.11 ms, 6 take 5.54; the training step 6 % faster).  Beyond 32 rounds a part of one is 3 %.  `wide`: the call may
// take that form.
inline int bwd_heads_of_group(int most, int left, int nblk, int nqblk, int shift_blocks, bool causal, bool wide) {
  if (left <= most) return left;
  if (!wide || !even_walks(nblk, nqblk, causal) || (long long)most * ((nblk + 3) / 4) > 32 * kCus) return most;
  auto time = [&](int heads) {
    if (heads == 0) return 0.0;
    const BwdEstimate t = bwd_estimate(heads, nblk, nqblk, shift_blocks, causal);
    return bwd_wide_is_faster(heads, nblk, nqblk, shift_blocks, causal) ? t.four : t.two;
  };
  int best = most;
  double least = 0.0;
  for (int h = most; h > most / 2 && h >= 1; h--) {
    const double t = left / h * time(h) + time(left % h);
    if (h == most || t < 0.99 * least) {
      least = t;
      best = h;
    }
  }
  return best;
}

// psi(dS) of a launch on its way from the backward to the dQ kernel.  While it fits the memory-side cache (256 MB) together with what the
// two kernels read and write beside it (codes of Q and K in two layouts and of dO, V and dO in bf16, three gradients), it is left to the
// caches.  From there on the dQ kernel loads it past them, and takes the last heads first, whose tiles were written last: the cache
// holds part of them.  Beyond 400 MB of psi(dS) that is little and displaces what the two kernels read again, so that
// sage_bwd_wide_kernel stores past the caches too (and the heads come in order).
// Whole steps, us, all through the caches -> loaded past them, last heads first, by MB in all (of them psi(dS); heads of N).
// d = 128, mask: 189 (129; 4 of 8192) 293 -> 294, 192 (42; 80 of 1024) 136 -> 140, 215 (28; 200 of 512) 146 -> 152, 218 (113; 14 of 4096)
// 275.1 -> 274.9, 243 (86; 42 of 2048) 218.7 -> 217.1, 250 (130; 16 of 4096) 293.5 -> 291.9, 266 (94; 46 of 2048) 226.5 -> 225.4,
// 283 (193; 6 of 8192) 448 -> 442, 288 (63; 120 of 1024) 215.7 -> 213.3, 302 (107; 52 of 2048) 251 -> 245, 360 (79; 150 of 1024) 264
// -> 262. d = 128, no mask: 188 (128; 8 of 4096) 250 -> 251, 206 (104; 26 of 2048) 207.6 -> 209.0, 230 (80; 80 of 1024) 220 -> 225,
// 237 (192; 3 of 8192) 420 -> 423, 248 (128; 32 of 2048) 230.7 -> 233.2, 277 (128; 16 of 1024 against 8192 keys) 259.0 -> 259.8, 279
// (144; 36 of 2048) 370 -> 368, 282 (192; 12 of 4096) 356 -> 354, 287 (100; 100 of 1024) 256.6 -> 255.8, 376 (256; 16 of 4096) 420
// -> 414, 496 (256; 64 of 2048) 477 -> 465. d = 64: mask 198 (161; 5 of 8192) 292 -> 295, 219 (79; 150 of 1024) 184 -> 186, 237
// (162; 20 of 4096) 268.5 -> 272.0, 252 (132; 64 of 2048) 223 -> 221, 277 (225; 7 of 8192) 349 -> 343, 293 (106; 200 of 1024) 234 ->
// 230, 315 (165; 80 of 2048) 276 -> 269; no mask 193 (100; 100 of 1024) 183 -> 185, 235 (160; 40 of 2048) 232.0 -> 232.7, 237 (192;
// 12 of 4096) 264 -> 272, 282 (192; 48 of 2048) 273 -> 268, 290 (150; 150 of 1024) 275 -> 273. Stored past the caches as well,
// steps, us: mask, 273 MB (32 of 4096) 488 -> 488.5, 382 (20 of 6144) 698 -> 696, 24 of 6144 819 -> 818, 545 (64 of 4096) 973 ->
// 973, 2164 (64 of 8192) 3514 -> 3485; no mask, 192 (12 of 4096) 354 -> 359, 256 (16 of 4096) 414 -> 420, 352 (22 of 4096) 697 ->
// 699, 512 (32 of 4096) 846 -> 844, 768 (12 of 8192) 1380 -> 1382, 1024 (16 of 8192) 1589 -> 1567.
// Not with few key blocks, whose short walks wait for their first loads.  d = 128, mask: 355 (27; 700 of 256) 213 -> 217, 377 (49; 350
// of 512) 254 -> 256, 415 (64; 300 of 640) 289 -> 292, 427 (76; 250 of 768) 298 -> 300, 410 (82; 200 of 896) 293.7 -> 293.1; no mask:
// 371 (43; 700 of 256) 231 -> 233, 379 (63; 450 of 384) 276 -> 279, 780 (195; 500 of 640) 600 -> 604, 491 (140; 250 of 768) 388 -> 387,
// 787 (225; 400 of 768) 586 -> 578; 628 (160; 64 of 8192 against 320 keys) 558 -> 567, 662 (250; 100 of 4096 against 640) 668 -> 676,
// 512 (256; 32 of 8192 against 1024) 547 -> 542.  d = 64: 360 (128; 64 of 8192 against 256) 292 -> 295, 394 (160; 64 of 8192 against
// 320) 354 -> 362, 412 (187; 300 of 1024 against 640) 370 -> 367, 400 (256; 64 of 4096 against 1024) 381 -> 364; 251 (87; 350 of 512)
// 206 -> 207, 292 (117; 300 of 640) 249 -> 247, 315 (140; 250 of 768) 284 -> 280; mask 399 (107; 500 of 640) 306.3 -> 306.9, 402 (121;
// 400 of 768) 312 -> 309.
struct DsTraffic {
  bool load_past, store_past;
};
inline DsTraffic ds_traffic(long long heads, int nblk, int nqblk, int shift_blocks, int d, bool causal) {
  long long tiles = (long long)nblk * nqblk;      // of a head
  if (causal) tiles = (long long)nqblk * (shift_blocks + 1) + (long long)nqblk * (nqblk - 1) / 2;
  const long long beside = 64ll * d * (7 * nqblk + 8 * nblk);
  const bool store_past = heads * tiles * 4096 >> 20 > 400;
  const bool load_past = heads * (tiles * 4096 + beside) >> 20 >= 250 && nblk >= (d == 64 ? 10 : causal ? 14 : 12);
  return {store_past || load_past, store_past};
}

// dQ with one Q block per workgroup and its waves on channel blocks (sage_bwd_dq_split_kernel; same bits): while the other form's
// workgroups, of two Q blocks each and three per CU, leave much of the machine idle, which walks of all lengths do longer than even
// ones: as long as the longest walk has 3.85 times the stages that one of its slots has on average.  On fuller machines this kernel
// is often still the faster, but the kernels around it in a training step get slower (32 heads of N = 2048: 30.7 -> 26.9, the
// backward before it 127.5 -> 131.7; 46 of 1024 against 3072 keys: 43.7 -> 45.9, 126.5 -> 136.8, the forward 57.7 -> 63.4), so the
// line lies where the whole step gains.  (Those run the same code with the same number of memory requests, and launched one at a
// time they take the same time with either form: it is not what the caches hold, and the chip's power limit would explain it.)
// Q blocks of all heads (N): step / dQ kernel, us, two Q blocks per workgroup -> one.
// With the mask, as many keys as queries, d = 128: 512 (2048) 124 / 28 -> 114 / 17, 752 (3000) 205 / 38 -> 197 / 27, 768 (2048) 159 / 29
// -> 155 / 22, 768 (6144) 369 / 72 -> 358 / 46; 799 (3000) 209.5 -> 210.3 (another time 211.8 -> 216.7), 880 (7000) 426 -> 422, 896
// (4096) 279.7 -> 279.8, 923 (4500) 393 -> 399, 960 (6144) 505 -> 512, 1024 (4096) 299 -> 304, 1136 (4500) 374 -> 379, 1248 (6144)
// 547 -> 550, 1312 (5200) 452 -> 458, 1476 (5200) 517 -> 506; d = 64: 640 (2500) 125 / 23 -> 120 / 17, 768 (2048) 110.5 / 20 ->
// 109.5 / 16, 1008 (1777) 117 -> 119, 1100 (7000) 407 -> 414, 1264 (5000) 306 -> 309. Walks of 112 blocks and more, twice: d = 128:
// 968 (7700) 485 -> 492, 1024 (8192) 533 -> 534, 1128 (12000) 879 -> 871, 1280 (8192) 737 / 155 -> 697 / 111, 1392 (7400) 660 ->
// 652, 1410 (9000) 892 -> 879, 1500 (16000) 1363 -> 1350, 1536 (8192) 765 / 152 -> 742 / 124, 2000 (16000) 1497 -> 1520; d = 64:
// 1024 (8192) 375 -> 371, 1280 (8192) 540 -> 511, 1504 (12000) 742 -> 746.
// More keys than queries: 1.1 times 640 (1024) 111 -> 108, 752 (1024) 126.5 -> 127.4, 726 (4224) 370 -> 374; 1.25 times 704 (2048)
// 194 -> 189.5; 1.5 times 544 (2048) 211 -> 200, 640 (2048) 213.5 -> 207.5, (1024) 131.8 -> 133.4 and at d = 64 95.3 -> 96.0, 726
// (4224) 473 -> 490; twice 462 (4224) 481 -> 464, 496 (1024) 141 -> 136, 594 (4224) 531 -> 541, 896 (8192) 1292 -> 1279; three times
// 416 (1024) 199 -> 193, 528 (1024) 240 -> 243, 594 (4224) 782 -> 800, 736 (1024) 269 -> 284. Without the mask: 512 (2048) 153 / 28
// -> 152 / 22.5, (4096) 264.5 / 49 -> 261.5 / 38.5, 640 (2048) 193 -> 199, (2500) 230.5 -> 236; d = 64: 672 (1777) 135.3 -> 138.
// One Q block a head leaves half of the other form idle at every size: 4000 heads of N = 64 329 / 40 -> 325 / 35.
inline bool use_dq_split(long long heads, int nblk, int nqblk, bool causal) {
  const long long blocks = heads * nqblk;
  if (nqblk == 1 || blocks <= 2 * kCus) return true;
  if (even_walks(nblk, nqblk, causal)) return false;
  const double slot = 0.5 * blocks * (nblk - 0.5 * nqblk) / (3 * kCus);
  return nblk >= (nqblk >= 112 ? 2.0 : 3.85) * slot;
}

}  // namespace sage
