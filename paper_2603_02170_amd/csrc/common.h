// Shared device-side types and helpers for the SageBwd kernels (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sage {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef unsigned short v8us __attribute__((ext_vector_type(8)));
typedef unsigned short v4us __attribute__((ext_vector_type(4)));

constexpr int kBlock = 64;  // B_q = B_kv: rows that share one quantisation scale

// ---------------------------------------------------------------------------
// Operand layouts written by the pre-pass.  Both cover a tensor X^ [N, d] of one
// head as consecutive 1 KiB fragments of 64 lanes x 16 bytes, so that a wave loads
// an MFMA operand with one 16-byte access per lane at `lane * 16`.
//
// F  ("row fragments", contraction over d):
//    fragment (rb, s), rb = 32-row block, s = 32-channel step; lane (r, h), r = lane % 32,
//    h = lane / 32, byte t:   X^[32 rb + r][32 s + 16 h + t]
// TF ("transposed fragments", contraction over rows):
//    fragment (rb, cb), cb = 32-channel block; lane (c, h), byte t = 4a + b:
//    X^[32 rb + 8a + 4h + b][32 cb + c]
//    The row order 8a + 4h + b is the order in which a 32x32 MFMA accumulator holds
//    its rows (register 4a + b of lane half h), so a quantised accumulator tile is
//    directly the matching operand of the next MFMA.
// Fragment index within a head: rb * (d / 32) + (s or cb).
// ---------------------------------------------------------------------------

__device__ __forceinline__ float bf16_bits_to_float(unsigned short u) {
  return __uint_as_float(((unsigned)u) << 16);
}

// round-to-nearest-even float -> bf16 bits (one conversion instruction for two values; NaN kept quiet)
__device__ __forceinline__ unsigned short float_to_bf16_bits(float f) {
  const __bf16 b = (__bf16)f;
  unsigned short u;
  __builtin_memcpy(&u, &b, 2);
  return u;
}

// max over the two 32-lane halves of a wave, result in every lane
__device__ __forceinline__ int half_swap_max_i32(int v) {
  auto r = __builtin_amdgcn_permlane32_swap((unsigned)v, (unsigned)v, false, false);
  int a = (int)r[0], b = (int)r[1];
  return a > b ? a : b;
}
__device__ __forceinline__ float half_swap_max_f32(float v) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float half_swap_sum_f32(float v) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// max over all 64 lanes of a NON-NEGATIVE float (result in every lane).  Non-negative floats
// order like their bit patterns, so the reduction runs on unsigned integers: four DPP steps
// inside each row of 16 lanes (the `old` value 0 is the identity of an unsigned max, which lets the
// compiler fold each lane permutation into the max instruction), then the row and half-wave swaps
// of gfx950.  No LDS traffic.
__device__ __forceinline__ float wave_max_nonneg_f32(float v) {
  unsigned u = __float_as_uint(v);
  unsigned t;
  t = (unsigned)__builtin_amdgcn_update_dpp(0, (int)u, 0xB1, 0xf, 0xf, false);   // quad_perm [1,0,3,2]
  u = u > t ? u : t;
  t = (unsigned)__builtin_amdgcn_update_dpp(0, (int)u, 0x4E, 0xf, 0xf, false);   // quad_perm [2,3,0,1]
  u = u > t ? u : t;
  t = (unsigned)__builtin_amdgcn_update_dpp(0, (int)u, 0x141, 0xf, 0xf, false);  // row_half_mirror
  u = u > t ? u : t;
  t = (unsigned)__builtin_amdgcn_update_dpp(0, (int)u, 0x140, 0xf, 0xf, false);  // row_mirror
  u = u > t ? u : t;
  auto r16 = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  u = r16[0] > r16[1] ? r16[0] : r16[1];
  auto r32 = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  u = r32[0] > r32[1] ? r32[0] : r32[1];
  return __uint_as_float(u);
}

// Loads and stores of what passes through once and does not fit the caches: they are told to let go of it first.  For whole 16-byte
// pieces of whole lines only: stores of 8 bytes that meet in the L2 otherwise, and loads of lines that another load takes the rest
// of, got slower (the backward of 36 heads of N = 1777, d = 64, 55 -> 83 us, a decoding step 73 -> 95).
template <class T>
__device__ __forceinline__ T stream_load(const T* p) {
  return __builtin_nontemporal_load(p);
}
template <class T>
__device__ __forceinline__ void stream_store(T* p, const T& v) {
  __builtin_nontemporal_store(v, p);
}

// INT32 sums that read as floats: accumulators that start from the bits of C0 = 1/(2 pi), an inline constant of the ISA, hold
// C0 + a 2^-26 exactly for |a| < 2^20 (see fwd_kernel.h).
constexpr int kBiasBits = 0x3E22F983;
constexpr float kBiasC0 = 0.15915494309189532f;
constexpr float kTwo26 = 67108864.0f;

// The product that starts a chain from B0.  As assembly, because the compiler folds the inline constant into one product
// only and makes a splat of 16 registers for several: with it the loop of sage_fwd_kernel formed the splat anew in every tile (8
// vector and 16 scalar instructions) and had no register to spare (256 and 17 parked; now 251; 16 heads of N = 8192 350 -> 337 us).
// The compiler does not see a matrix instruction here, so the waits around one are written out: two states after a vector write of
// an operand, two before the next product of the chain reads the result as its C, which must be the only thing that ever reads it (a
// copy or a spill in between would read an unfinished result), and the result is kept off its operands' registers, as the compiler
// keeps those of its own products of this size.  A test reads both from the assembly of the build.
__device__ __forceinline__ v16i mfma_from_bias(const v4i& a, const v4i& b) {
  v16i d;
  asm("s_nop 1\n\tv_mfma_i32_32x32x32_i8 %0, %1, %2, 0.15915494\n\ts_nop 1" : "=&v"(d) : "v"(a), "v"(b));
  return d;
}

typedef const __attribute__((address_space(1))) void* gptr_t;
typedef __attribute__((address_space(3))) void* lptr_t;

// One 16-byte piece per lane, global -> LDS, no registers in between.  The LDS address is
// `lds_base + lane * 16` (the hardware adds the lane offset to the wave-uniform base).
__device__ __forceinline__ void async_copy_16(const void* gsrc_lane, void* lds_base) {
  __builtin_amdgcn_global_load_lds((gptr_t)gsrc_lane, (lptr_t)lds_base, 16, 0, 0);
}
__device__ __forceinline__ void async_copy_4(const void* gsrc_lane, void* lds_base) {
  __builtin_amdgcn_global_load_lds((gptr_t)gsrc_lane, (lptr_t)lds_base, 4, 0, 0);
}

// A wave-uniform address as the compiler must take it: in scalar registers, so that an access adds 32 bits of lane offset to it
// (left alone it keeps 64-bit sums of base and lane in vector registers).
typedef __attribute__((address_space(1))) char* gbytes_t;
__device__ __forceinline__ gbytes_t uniform(const void* p) {
  gbytes_t g = (gbytes_t)p;
  asm("" : "+s"(g));
  return g;
}
// Two 16-byte pieces per lane to base + lane_offset and OFFSET behind it, past the caches (as stream_store does) where `stream` is
// not 0.  The branch is inside the assembly, as below, and the compiler would make one plain store of both sides.  It does not see
// stores here: the wait states in front are for a base that a vector instruction wrote, the one behind for an overwrite of the data,
// and a wait for them has to be written out.
template <int OFFSET>
__device__ __forceinline__ void store_pair(gbytes_t base, unsigned lane_offset, const v4i& a, const v4i& b, int stream) {
  asm volatile(
      "s_nop 4\n\ts_cmp_eq_u32 %4, 0\n\ts_cbranch_scc1 .Lkeep%=\n\t"
      "global_store_dwordx4 %0, %1, %3 nt\n\tglobal_store_dwordx4 %0, %2, %3 offset:%5 nt\n\ts_branch .Ldone%=\n"
      ".Lkeep%=:\n\tglobal_store_dwordx4 %0, %1, %3\n\tglobal_store_dwordx4 %0, %2, %3 offset:%5\n"
      ".Ldone%=:\n\ts_nop 1" ::"v"(lane_offset), "v"(a), "v"(b), "s"(base), "s"(stream), "n"(OFFSET)
      : "scc", "memory");
}
__device__ __forceinline__ void copy_16(gbytes_t gsrc_lane, void* lds_base) {
  __builtin_amdgcn_global_load_lds((gptr_t)gsrc_lane, (lptr_t)lds_base, 16, 0, 0);
}
__device__ __forceinline__ void copy_4(gbytes_t gsrc_lane, void* lds_base) {
  __builtin_amdgcn_global_load_lds((gptr_t)gsrc_lane, (lptr_t)lds_base, 4, 0, 0);
}

// Issue priority P for waves 4 to 7 of a workgroup of eight: where two waves share a SIMD the arbiter favours the older one.
// (The branch is inside the assembly: the code around it stays one basic block for the scheduler and the register allocator.)
template <int P>
__device__ __forceinline__ void first_for_younger_waves(int wave) {
  asm volatile("s_cmp_lt_u32 %0, 4\n\ts_cbranch_scc1 .Lolder%=\n\ts_setprio %1\n.Lolder%=:" ::"s"(wave), "n"(P) : "scc");
}

// A wave-uniform value through the scalar cache: no vector-memory instruction and no register of 64 lanes.  (The
// buffer must not be written by the same kernel.)
__device__ __forceinline__ float scalar_load(const float* p) {
  return *(const __attribute__((address_space(4))) float*)(uintptr_t)p;
}

// Two neighbours.
__device__ __forceinline__ v2f scalar_load2(const float* p) {
  typedef v2f v2f_dword __attribute__((aligned(4)));
  return *(const __attribute__((address_space(4))) v2f_dword*)(uintptr_t)p;
}

// Immediate of `s_waitcnt vmcnt(n)` alone (the LDS / scalar and export counters are left at their
// maxima = no wait): the six bits of n sit in bits 3:0 and 15:14.
constexpr int vmcnt_only(int n) { return 0x0F70 | (n & 15) | ((n >> 4) << 14); }
// Keeps memory operations in program order across this point (for the compiler; no instruction).
__device__ __forceinline__ void compiler_fence() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// Workgroup barrier that waits for this wave's LDS traffic only.  (__syncthreads() would
// also drain the asynchronous global->LDS copies that are meant to stay in flight.)
__device__ __forceinline__ void barrier_lds_only() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}
// Same, after all of this wave's global-memory operations (the async copies included).
__device__ __forceinline__ void barrier_all_memory() {
  __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0), as a builtin so the compiler's own wait tracking sees it
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Where row n of head bh = b * H + h of one of the caller's [.., N, d] tensors starts, in elements:
// dense [B, H, N, d] has strides (H N d, N d, d), token-major [B, N, H, d] has (N H d, d, H d).
struct RowView {
  size_t batch_stride, head_stride, row_stride;
  int H;
  __host__ __device__ size_t row(int bh, size_t n) const {
    return (size_t)(bh / H) * batch_stride + (size_t)(bh % H) * head_stride + n * row_stride;
  }
};

// Workgroup id -> (head, work item of the head).  Consecutive ids go round-robin over the 8 XCDs, so
// with a multiple of 8 heads every head's workgroups are given one XCD and share its L2.  The heads of
// an XCD are taken `head_set` at a time, and inside such a set the items go heaviest first over ALL its
// heads (item 0 of every head, then item 1, ...): with the causal mask the last workgroups to start
// are then the lightest of several heads, not of one.  That shortens the tail of short-sequence
// launches (13 % of the step at N = 2048); from more than 32 items a head on the forward and the backward with two KV blocks
// per workgroup lose 2 % to it (several heads' operands compete for the L2), so they take one head at a time there.
// Other head counts are laid out densely over the XCDs: no workgroup is without work (it would still queue for a whole
// workgroup's LDS and wave slots before it could exit) and a single head spreads over all XCDs instead of one.
// Short sequences take the items heaviest first over ALL heads (head after head, the heaviest items of the
// last heads start last: the backward of 36 heads of N = 1777 took half as long again as its work), longer ones over
// sets of up to four heads, as above.
struct WorkItem {
  int head, item;
};
// > 0: that many heads of an XCD per set; < 0: the dense layout, sets of that many heads (on a machine of one XCD, so to
// speak, so that the mapping below stays one formula).  A set divides the heads evenly; where four do not divide an XCD's heads,
// short sequences take the largest number up to eight that does (five heads one at a time left the last head's heaviest items to the end:
// calls with the mask, forward and backward in us, 40 heads of N = 1024 43 + 90 -> 39 + 65, of 2048 84 + 196 -> 73 + 167, 56 of 4096
// 276 + 808 -> 258 + 764; nine heads have sets of three).  Where that is one or two, all of them, up to 31 heads and 768 items: 152
// heads (19) of N = 512 55 + 100 -> 48 + 70, 248 (31) of 1024 163 + 381 -> 154 + 287; larger sets crowd the L2 (34 heads in sets of
// two -> all: N = 1024 164 + 323 -> 170 + 317, 2048 403 + 945 -> 421 + 980; 37 one at a time -> all: 1024 190 + 407 -> 188 + 341,
// 2048 451 + 1084 -> 458 + 1064; 31 of 32 items, d = 64 and N = 2048, backward 667 -> 686).
__host__ __device__ inline int head_set_for(int items, int heads, bool always = false) {
  const bool dense = heads % 8 != 0;
  const int pool = dense ? heads : heads / 8;
  int hs = dense && items <= 32 ? pool : (always || dense || items <= 32) ? 4 : 1;
  if (items <= 32 && pool % hs != 0 && pool > hs) {
    hs = 8;
    while (pool % hs != 0) hs--;
    if (hs < 3 && pool < 32 && pool * items <= 768) hs = pool;
  }
  while (pool % hs != 0) hs--;
  return dense ? -hs : hs;
}
// The grid is heads * items workgroups, each of which has a (head, item) of its own (a test goes through them on the host): a
// kernel needs no check of its head, and without one the loads of its arguments need not wait for the mapping.
__host__ __device__ inline int grid_for(int heads, int items) { return heads * items; }
__host__ __device__ inline WorkItem work_item(int block, int items, int head_set) {
  const int xcds = head_set < 0 ? 1 : 8, hs = head_set < 0 ? -head_set : head_set;
  const int xcd = block % xcds, slot = block / xcds;
  const int hset = slot / (items * hs), rem = slot % (items * hs);
  return WorkItem{xcd + xcds * (hset * hs + rem % hs), rem / hs};
}

// Which of a launch's workgroups share a CU, for kernels of which two or more fit one.  The first of an XCD go round its 32
// CUs, heaviest first, so that a CU's second workgroup is its 33rd: with the mask the CU with the heaviest first one gets the
// heaviest second one too, and a launch of about one round takes as long as that CU.  The second 32 (up to `end`) in reverse
// order give every CU about the same.  us, heaviest first -> this way: forward, 32 heads of N = 2048 44.6 -> 42.4 (blocks of
// 128), 64 of 1024 29.1 -> 26.0, 8 of 8192 134 -> 123, 9 of 7000 119 -> 107; d = 64, 36 of 1777 28.6 -> 27.1, 12 of 8192 158 ->
// 118; backward, d = 64 (sage_bwd_single_kernel), 10 of 3000 64.5 -> 56.0, 6 of 4096 71.0 -> 68.3, 36 of 1777 56.7 -> 55.5; the
// sweep for the maxima of blocks of 128 queries with the sweep behind it, 32 of 2048 126.2 -> 124.3, the whole step 225.3 ->
// 221.7, 24 of 1700 174 -> 165.
__host__ __device__ inline int folded(int block, int end) {
  const int slot = block >> 3;
  return slot >= 32 && slot < end ? (32 + end - 1 - slot) << 3 | (block & 7) : block;
}
// Up to `rounds` times the CUs, and some more where walks are long (forward, us: 12 heads of N = 6000, 564 workgroups, 104 ->
// 100.5; d = 64, 24 of 4096, 768, 62.2 -> 59.3, but 64 of 1500, 768, 31.2 -> 32.1); launches of several rounds give out their
// workgroups as CUs get free.  So does one of a kernel that has a CU to itself (per_cu = 1): the lightest of the first 32 is
// done first and has to get the heaviest of the second (backward of d = 64 with Q-smoothing, us, this way -> heaviest first: 16
// heads of N = 2048 57.5 -> 47.6, 8 of 4096 98.5 -> 80.5, 32 of 1024 36.3 -> 30.9, 40 of 700 28.5 -> 24.8).
__host__ __device__ inline int fold_end(int grid, int items, int rounds, int per_cu) {
  if (per_cu < 2 || grid <= 256 || grid > (items >= 24 && rounds < 3 ? 3 : rounds) * 256) return 0;
  return grid / 8 < 64 ? grid / 8 : 64;
}

// Both that order and a kernel with a CU to itself whose second round is to be the lighter one count on the heaviest items being the
// first of the whole launch, which sets of heads do not give: where a set begins, its heaviest items follow the lightest of the one
// before, and in the last round they end the launch.  Such launches take the items heaviest first over all heads (of an XCD, or of
// the call in the dense layout); few as their workgroups are, their heads do not crowd the L2.  us, in sets -> over all heads:
// forward (four waves per 32 queries), 7 heads of N = 4096 77.0 -> 50.2 (two waves 59.2), 5 of 6144 91.4 -> 66.1 (79.2), 5 of 8192
// 133.4 -> 110.1 (127.3), 9 of 3000 49.5 -> 42.9 (48.3); forward, 7 of 7000 131 -> 110.6 (not folded 127), 11 of 7000 157.6 -> 135.5
// (152.8); d = 64, 11 of 7000 125 -> 97.5 (115.5); training steps, d = 64, 5 of 5000 195 -> 161 (173), 10 of 4096 193 -> 165 (185),
// 7 of 7000 345 -> 275 (333).
__host__ __device__ inline int all_heads(int heads) { return heads % 8 != 0 ? -heads : heads / 8; }
struct LaunchOrder {
  int head_set, fold_end;
};
__host__ __device__ inline LaunchOrder folded_order(int heads, int items, int rounds, int per_cu) {
  const int end = fold_end(grid_for(heads, items), items, rounds, per_cu);
  return {end != 0 ? all_heads(heads) : head_set_for(items, heads), end};
}
// sage_fwd_quad_kernel under the mask: more than one round of one workgroup per CU (see use_fwd_quad)
__host__ __device__ inline int quad_head_set(int heads, int items) {
  return grid_for(heads, items) > 256 ? all_heads(heads) : head_set_for(items, heads);
}

// What a workgroup of a pre-pass launch takes: a job, a head, a block (or chunk) of its rows.  The grid is (blocks, heads, jobs), whose
// ids, and so a head's blocks, go round the 8 XCDs; or, `own_xcd`, (8, blocks, jobs x heads / 8), in which a head's workgroups have
// one XCD, the same in every launch and the one that the attention kernels give the head: what one launch has read or written is then
// in the L2 that the next one reads through (see prepass_own_xcd).  The grid holds what a workgroup needs for it, so that it divides by
// nothing, and the kernels are instantiated for either: a workgroup that has to look in the arguments which of the two it is begins to
// load that much later (0.3 us a launch of the quantiser, whose job lies at a place that waits for the number of heads; decoding, 32
// heads of 4096 keys, 28.6 us, with the choice at run time 29.2; sage_fwd_short_kernel has it at run time all the same).
struct PrepassItem {
  int job, head, block;
};
__host__ __device__ inline PrepassItem prepass_item(int x, int y, int z, bool own_xcd, int heads) {
  if (!own_xcd) return PrepassItem{z, y, x};
  int job = 0, group = z;
  for (; group >= heads / 8; group -= heads / 8) job++;
  return PrepassItem{job, x + 8 * group, y};
}
// The last rows of the heads of each XCD first: the order in which an L2 that does not hold all of it has kept what the launch before has
// read of K (kmean_partial_kernel), or written of O (the forward, where the backward's pre-pass quantises dO alone).
__host__ __device__ inline PrepassItem last_rows_first(const PrepassItem& i, int blocks, int heads) {
  return PrepassItem{i.job, heads - 8 + 2 * (i.head & 7) - i.head, blocks - 1 - i.block};
}
inline dim3 prepass_grid(int blocks, int heads, int jobs, bool own_xcd) {
  return own_xcd ? dim3(8, blocks, jobs * (heads / 8)) : dim3(blocks, heads, jobs);
}

// Row of K or V that a load of sage_fwd_decode_kernel for row `row` reads: a row that does not exist re-reads the last one that does
// (which changes no maximum of its block), and all rows of a block that is not the wave's (`mine` false: the load ahead of a wave's
// last block) are one row.  The loop stays without a branch, and no block is read twice (two sequences of 32 heads of 8192 keys,
// where that was an eighth of all reads: 75.5 us a call -> 73.0 with Q's fragments in LDS).
__host__ __device__ inline int decode_row(int row, bool mine, int nk) {
  const int last = mine ? nk - 1 : 0;
  return row < last ? row : last;
}

}  // namespace sage
