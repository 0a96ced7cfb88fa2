// Pre-pass kernels: K-smoothing mean, optional Q-smoothing block mean, the per-block
// INT8 quantiser psi, delta = rowsum(dO o O), and the export (inspection) kernels.
//
// Paper: Sec. 3 "Quantization" (X^ = round(X / delta_X), delta_X = max|X| / 127),
// Sec. 3 "Q and K Smoothing" (mu_K over the whole key tensor, mu_Qi per block),
// Algorithm 1 "Quantization" line, Algorithm 2 line 2 (D) and line 6 (psi(dO_i)).
//
// The stored INT8 codes and FP32 scales are a bit-exact contract, so the arithmetic
// here is fixed: mean = (float64 sum) / N rounded once to FP32; x - mu in FP32;
// a = max|x|; s = a / 127 and r = 127 / a as IEEE FP32 divisions; q = rne(x * r).
#pragma once

#include <type_traits>

#include "common.h"

namespace sage {

#pragma clang fp contract(off)

// Rows of K per workgroup of the mean reduction: the host picks the largest of these that still gives
// the launch a few workgroups per CU (the consumer sums one partial per chunk and channel).
inline int mean_chunk_rows(int heads, int N) {
  int rows = 1024;
  while (rows > 128 && (long long)heads * ((N + rows - 1) / rows) < 1024) rows >>= 1;
  return rows;
}

// ---- QK-norm fused into the pre-pass (paper Sec. 4, "Stabilizing Outliers with QK-Norm") ----------
// y = x / sqrt(mean_c x^2 + eps) * gamma per token, rounded to bf16: the tensor a bf16 model hands to the
// attention, so the fused pre-pass gives the bits of "normalise, then quantise".  Arithmetic (part of the
// bit-exact contract): sum of squares in float64 (exact for bf16 inputs), r = 1 / sqrt(sum / D + eps) in
// float64 rounded once to FP32, y = bf16((x *_f32 r) *_f32 gamma).
struct QkNorm {
  const float* gamma;   // [D] per-channel gain, or nullptr: no normalisation
  float eps;
};
__device__ __forceinline__ float qknorm_rscale(double sumsq, int D, float eps) {
  return (float)(1.0 / sqrt(sumsq / (double)D + (double)eps));
}
__device__ __forceinline__ float qknorm_apply(float x, float r, float g) {
  return bf16_bits_to_float(float_to_bf16_bits((x * r) * g));
}

// Float64 column sums of `rows` rows at `base`, over the 256 threads of a workgroup: thread t adds the rows
// t / TPR, t / TPR + RPP, ... of its 8 channels 8 (t % TPR) .. into acc.
// (bf16 data of ordinary range sum exactly in float64, so the result does not depend on the order.)
// NORMED: of the normalised rows, that many of a thread's rows at a time (0: of the rows as they are).  Kernels are instantiated for
// each, since the normalising loop takes registers that the plain one's occupancy needs (quantiser with the mean inside at d = 128
// 136 for 87, three waves per SIMD for five; forward calls, us, both loops in one kernel -> apart: 1000 heads of N = 64 31.6 -> 30.5,
// 300 of 128 25.2 -> 23.7, blocks of 128, d = 64, 1000 of 64 21.2 -> 19.2).
template <int D, int NORMED>
__device__ __forceinline__ void column_sums(const unsigned short* __restrict__ base, const size_t row_stride, const int rows,
                                            const QkNorm& norm, double (&acc)[8]) {
  constexpr int TPR = D / 8;          // threads per row, 8 channels (16 bytes) each
  constexpr int RPP = 256 / TPR;      // rows per pass
  const int t = threadIdx.x;
#pragma unroll
  for (int e = 0; e < 8; e++) acc[e] = 0.0;
  const int tr = t / TPR, tc = t % TPR;
  if constexpr (NORMED > 0) {
    // the mean is taken over the normalised keys: the TPR threads of a row share its sum of squares
    static_assert(NORMED == 1 || NORMED == 4, "one row, or four");
    float g[8];
#pragma unroll
    for (int e = 0; e < 8; e++) g[e] = norm.gamma[tc * 8 + e];
    // Four rows at a time: their loads, sums and shuffles overlap, and a thread takes the float64 root and quotient of one of them
    // for its neighbours.  (One row after the other, with every thread of a row taking its root, the loop is one chain, which heads
    // of one block are as well off with, in two thirds of the registers.  Forward calls, us, one -> four: 8 heads of N = 269 21.6 ->
    // 19.0, 8 of 4163 79.3 -> 77.5, 64 of 8192 838 -> 834, 8 of 512 32.1 -> 25.6; training step of 32 heads of 2048 187.1 -> 183.2;
    // but 1000 of 64 34.7 -> 37.3, blocks of 128, d = 64, 21.6 -> 25.1, 400 of 64 12.9 -> 14.1.)
    const int lane = t & 63;
    for (int r0 = 0; r0 < rows; r0 += NORMED * RPP) {  // whole passes: the shuffles need every lane
      v8us v[NORMED];
      double ss[NORMED];
#pragma unroll
      for (int u = 0; u < NORMED; u++) {
        v[u] = v8us{0, 0, 0, 0, 0, 0, 0, 0};
        if (r0 + u * RPP + tr < rows) v[u] = *(const v8us*)(base + (size_t)(r0 + u * RPP + tr) * row_stride + tc * 8);
      }
#pragma unroll
      for (int u = 0; u < NORMED; u++) {
        ss[u] = 0.0;
#pragma unroll
        for (int e = 0; e < 8; e++) {
          const float x = bf16_bits_to_float(v[u][e]);
          ss[u] += (double)(x * x);
        }
      }
#pragma unroll
      for (int off = 1; off < TPR; off <<= 1)
#pragma unroll
        for (int u = 0; u < NORMED; u++) ss[u] += __shfl_xor(ss[u], off, 64);
      double own = ss[0];
      if constexpr (NORMED == 4) own = (tc & 2) ? ((tc & 1) ? ss[3] : ss[2]) : ((tc & 1) ? ss[1] : ss[0]);
      const float mine = qknorm_rscale(own, D, norm.eps);
#pragma unroll
      for (int u = 0; u < NORMED; u++) {
        __builtin_amdgcn_sched_barrier(0);      // (row after row: side by side they cost up to 22 registers)
        const float rs = NORMED == 1 ? mine : __shfl(mine, (lane & ~(TPR - 1)) + u, 64);
        if (r0 + u * RPP + tr < rows) {
#pragma unroll
          for (int e = 0; e < 8; e++) acc[e] += (double)qknorm_apply(bf16_bits_to_float(v[u][e]), rs, g[e]);
        }
      }
    }
  } else {
    int r = tr;
    // four independent 16-byte loads in flight per thread
    for (; r + 3 * RPP < rows; r += 4 * RPP) {
      v8us v[4];
#pragma unroll
      for (int u = 0; u < 4; u++) v[u] = *(const v8us*)(base + (size_t)(r + u * RPP) * row_stride + tc * 8);
#pragma unroll
      for (int u = 0; u < 4; u++)
#pragma unroll
        for (int e = 0; e < 8; e++) acc[e] += (double)bf16_bits_to_float(v[u][e]);
    }
    for (; r < rows; r += RPP) {
      v8us v = *(const v8us*)(base + (size_t)r * row_stride + tc * 8);
#pragma unroll
      for (int e = 0; e < 8; e++) acc[e] += (double)bf16_bits_to_float(v[e]);
    }
  }
}

// ---- K mean, stage 1: float64 column sums of a chunk of rows -----------------------
// Stage 2, the sum over the chunks, the division by N and the one rounding to
// FP32, runs at the start of every workgroup that quantises a block of K (prepass_quant_kernel).
template <int D, int NORMED, bool OWN_XCD = false>
__global__ void __launch_bounds__(256) kmean_partial_kernel(const unsigned short* __restrict__ K, RowView view,
                                                            double* __restrict__ kpart, int N,
                                                            int nchunk, int chunk_rows, QkNorm norm, int heads) {
  constexpr int TPR = D / 8;
  constexpr int RPP = 256 / TPR;
  __shared__ double red[256][8];
  const int t = threadIdx.x;
  const PrepassItem item = prepass_item(blockIdx.x, blockIdx.y, blockIdx.z, OWN_XCD, heads);
  const int chunk = item.block, bh = item.head;
  const int row0 = chunk * chunk_rows;
  double acc[8];
  column_sums<D, NORMED>(K + view.row(bh, row0), view.row_stride, min(chunk_rows, N - row0), norm, acc);
#pragma unroll
  for (int e = 0; e < 8; e++) red[t][e] = acc[e];
  __syncthreads();
  if (t < D) {
    double s = 0.0;
    if (N <= 2 * kBlock) {
      // (in the order in which the quantiser adds the groups of a head that it sums itself: short heads have one mean in all forms, also
      // where their sums are not exact)
      for (int g = 0; g < RPP; g += RPP / 4) {
        double w[RPP / 4];
#pragma unroll
        for (int k = 0; k < RPP / 4; k++) w[k] = red[(g + k) * TPR + t / 8][t % 8];
#pragma unroll
        for (int off = 1; off < RPP / 4; off <<= 1)
#pragma unroll
          for (int k = 0; k < RPP / 4; k += 2 * off) w[k] += w[k + off];
        s += w[0];
      }
    } else {
      for (int g = 0; g < RPP; g++) s += red[g * TPR + t / 8][t % 8];
    }
    kpart[((size_t)bh * nchunk + chunk) * D + t] = s;
  }
}

// The chunk sums of a head, added by the 256 threads of a workgroup into red[256 / D][D] (whose rows the reader adds in
// order): thread t takes channel t % D of every (256 / D)-th chunk, eight loads in flight.  The sum stands before all else
// that a workgroup does with K, and each load waits for an L2 hit: with D threads adding one chunk after the other, a forward of 512
// queries against 4096 keys, 32 heads, d = 128 took 67.3 us, this way 61.4.
template <int D>
__device__ __forceinline__ void head_sums(const double* __restrict__ part, const int nchunk, double* red) {
  constexpr int GROUPS = 256 / D;
  const int t = threadIdx.x;
  part += t % D;
  double s = 0.0;
  int k = t / D;
  for (; k + 7 * GROUPS < nchunk; k += 8 * GROUPS) {
    double v[8];
#pragma unroll
    for (int u = 0; u < 8; u++) v[u] = part[(size_t)(k + u * GROUPS) * D];
#pragma unroll
    for (int u = 0; u < 8; u++) s += v[u];
  }
  for (; k < nchunk; k += GROUPS) s += part[(size_t)k * D];
  red[t] = s;
  __syncthreads();
}

// Short heads are summed by every workgroup that quantises a block of K, each for itself, without the launch of stage 1:
// what that launch costs (about 2 us) against what one workgroup reads (N * D) and what all of them read.  Forward calls,
// us without -> with: 1 head, d = 128, N = 512: 17.8 -> 17.4, 768: 20.9 -> 21.2; in millions of elements read by all, 64
// heads of 256 (8.4): 18.5 -> 17.2, 64 of 320 (13.1): 20.0 -> 19.8, 32 of 512 (16.8): 21.7 -> 22.1, 128 of 384 (38): 31.9 ->
// 37.2, 128 of 512 (67): 37.9 -> 49.6; d = 64, 48 of 512 (12.6): 18.8 -> 18.2, 128 of 384 (18.9): 23.6 -> 24.4.
inline bool mean_inline(int heads, int N, int D) {
  return (long long)N * D <= 65536 && (long long)heads * ((N + kBlock - 1) / kBlock) * N * D <= (14 << 20);
}

// The rounding of psi on values held as FP32: q = rne(x * r) clamped to +-127 (which matters where r = 127 / max|x|
// overflows, blocks of the smallest numbers, and for NaN: both become codes), four packed into a register.  x * r is rounded to FP32
// before the addition that takes it to an integer, so the codes are those of rintf.  Without CLAMP: where neither can be.
template <bool CLAMP = true>
__device__ __forceinline__ int quantise_4(const float x0, const float x1, const float x2, const float x3, const float r) {
#pragma clang fp contract(off)
  const float x[4] = {x0, x1, x2, x3};
  unsigned u[4];
#pragma unroll
  for (int e = 0; e < 4; e++) {
    const float y = CLAMP ? __builtin_amdgcn_fmed3f(x[e] * r, -127.f, 127.f) : x[e] * r;
    u[e] = __float_as_uint(y + 12582912.0f);               // 1.5 * 2^23: rne(y) in the low mantissa bits
  }
  return (int)(__builtin_amdgcn_perm(u[1], u[0], 0x0c0c0400u) | __builtin_amdgcn_perm(u[3], u[2], 0x04000c0cu));
}
template <bool CLAMP = true>
__device__ __forceinline__ v4i quantise_16(const float (&x)[16], const float r) {
  v4i o;
#pragma unroll
  for (int w = 0; w < 4; w++) o[w] = quantise_4<CLAMP>(x[4 * w], x[4 * w + 1], x[4 * w + 2], x[4 * w + 3], r);
  return o;
}

// ---- psi on one 64-row block (of a numerics block of 64 or 128 rows) -------------
struct QuantJob {
  const unsigned short* src;   // bf16, rows addressed through `view`
  RowView view;                // where the rows of src (and of O) lie in the caller's tensor
  int N, Np;                   // rows of src that exist; rows of the workspace tensors (N rounded up to 64)
  int q_like;                  // host side only: a Q-like tensor (numerics blocks of B_q rows) or a K-like one (B_kv)
  int8_t* outF;                // F layout or nullptr
  int8_t* outTF;               // TF layout or nullptr
  float* scale;                // [BH, N/64]
  const double* mean_part;     // K-smoothing: float64 column sums [BH, nchunk, D] of the whole head; the
                               // mean (sum / N, rounded once to FP32) is subtracted from every row.  Else nullptr
  int nchunk;
  int mean_inline;             // K-smoothing of a short head: no chunk sums, the workgroup sums the head itself
  float* mu_head_out;          // [BH, D]: where block 0 of each head stores that mean
  float* mu_block_out;         // [BH, N/64, D]: if set, the block mean is computed, stored and subtracted
  const unsigned short* O;     // bf16 [BH, N, D] or nullptr: delta = rowsum(src o O)
  float* delta;                // [BH, N]: -rowsum(src o O)
  const float* lse;            // [BH, N] or nullptr: nl2 = -lse * log2(e) for the backward
  float* nl2;                  // [BH, N]
  QkNorm norm;                 // QK-norm applied to src before anything else (Q and K jobs), or gamma == nullptr
  unsigned short* norm_out;    // if set: the normalised rows as dense bf16 [BH, Np, D] (for the Q-smoothing bias)
};
// Arguments of a launch, and of one with an XCD for every head, whose workgroups need the number of heads before anything else.  (In
// front of the jobs there, with them not moved here: two queries against 320 keys of 54 heads, d = 64, 13.6 us, with eight bytes in front
// 13.8; 64 heads of N = 256 15.3, with the numbers behind the jobs 15.6.)
struct QuantJobs {
  QuantJob job[4];
};
struct OwnXcdJobs {
  int blocks, heads;           // of every job's workgroups
  QuantJob job[4];
};

// Per job: N = rows of the caller's tensor, Np = N rounded up to a multiple of 64 = rows of its workspace
// tensors (Q-like and K-like tensors may have different lengths).  Rows N .. Np-1 do not exist: they are
// read as zeros AFTER the smoothing (so they change no absmax), enter no mean, get delta = 0 and
// -L*log2(e) = -inf (P = 0 in the backward).  The grid's x extent covers the longest job.
//
// SUB = 64-row blocks per numerics block (Algorithm 1 leaves B_q, B_kv free): 1, or 2 for blocks of 128 rows.
// A workgroup takes one numerics block; its scale (and block mean) is stored once per 64-row block: the
// attention kernels index scales, means and bias rows by 64-row block whatever the numerics block is.
// MEAN: the K job adds chunk sums, or sums its head itself (jobs of a short K; instantiations of their own, since the summing
// loops cost the registers that the others' occupancy needs), or sums the normalised rows of its head, four at a time or
// one (see normed_rows_by_fours).
enum : int { kMeanOfChunks, kMeanInline, kMeanInlineNormed, kMeanInlineNormedBlock };
// Waves per SIMD (left to itself the compiler takes 119 registers for plain keys where 87 do).
constexpr int quantiser_waves(int D, int SUB, int mean) {
  return mean == kMeanOfChunks ? 1 : mean == kMeanInlineNormed || SUB * D > 128 ? 3 : 5;
}
template <int D, int SUB, int MEAN, bool OWN_XCD = false>
__global__ void __launch_bounds__(256, quantiser_waves(D, SUB, MEAN)) prepass_quant_kernel(std::conditional_t<OWN_XCD, OwnXcdJobs, QuantJobs> jobs) {
  constexpr bool INLINE_MEAN = MEAN != kMeanOfChunks;
  constexpr int ROWS = SUB * kBlock;
  constexpr int CPR = D / 16;            // 16-channel chunks per row
  constexpr int NCH = ROWS * CPR / 256;  // chunks per thread
  constexpr int NTF = ROWS / 16 * D / 256;   // TF chunks per thread
  static_assert(SUB == 1 || SUB == 2, "numerics blocks of 64 or 128 rows");
  __shared__ __attribute__((aligned(16))) int8_t tile[ROWS * D];
  __shared__ __attribute__((aligned(16))) float colbuf[64 * D / 4];   // used by the block mean only (16 rows at a time)
  __shared__ float mu_s[D];
  __shared__ double sumsq[ROWS];         // QK-norm: the rows' sums of squares, then their factors
  __shared__ float wmax[4];

  PrepassItem item{(int)blockIdx.z, (int)blockIdx.y, (int)blockIdx.x};
  if constexpr (OWN_XCD) {
    item = prepass_item(blockIdx.x, blockIdx.y, blockIdx.z, true, jobs.heads);
    // (job 0: K where there are chunk sums, or dO alone)
    if (MEAN == kMeanOfChunks && item.job == 0) item = last_rows_first(item, jobs.blocks, jobs.heads);
  }
  const QuantJob jb = jobs.job[item.job];
  const int t = threadIdx.x;
  const int blk = item.block * SUB, bh = item.head;                         // first 64-row block
  const int N = jb.N, Np = jb.Np;
  const RowView view = jb.view;
  const int nblk = Np / kBlock;
  if (blk >= nblk) return;
  const int nsub = min(SUB, nblk - blk);                                    // 64-row blocks of the workspace here
  const size_t tile_off = view.row(bh, (size_t)blk * kBlock);               // in the caller's tensors
  const int rows_here = min(ROWS, N - blk * kBlock);                        // rows of this block that exist

  // the rows as FP32, 16 channels per chunk: chunk c = t + 256 it is (row c / CPR, channels 16 (c % CPR) ..)
  float x[NCH][16];
#pragma unroll
  for (int it = 0; it < NCH; it++) {
    const int c = t + 256 * it;
    const int row = c / CPR, ch = c % CPR;
    v8us lo = {0, 0, 0, 0, 0, 0, 0, 0}, hi = {0, 0, 0, 0, 0, 0, 0, 0};
    if (row < rows_here) {
      const unsigned short* p = jb.src + tile_off + (size_t)row * view.row_stride + ch * 16;
      lo = *(const v8us*)p;
      hi = *(const v8us*)(p + 8);
    }
#pragma unroll
    for (int e = 0; e < 8; e++) {
      x[it][e] = bf16_bits_to_float(lo[e]);
      x[it][8 + e] = bf16_bits_to_float(hi[e]);
    }
  }

  if (jb.norm.gamma != nullptr) {
    // QK-norm: the CPR threads of a row (consecutive lanes) form its sum of squares; one thread per row then takes
    // the float64 root and quotient (in every thread of the row they cost more than all the rest of this kernel:
    // B2 H16 N2048 d128 with blocks of 128, 57 us before, and the partner block was normalised twice)
#pragma unroll
    for (int it = 0; it < NCH; it++) {
      const int c = t + 256 * it;
      double ss = 0.0;
#pragma unroll
      for (int e = 0; e < 16; e++) ss += (double)(x[it][e] * x[it][e]);
#pragma unroll
      for (int off = 1; off < CPR; off <<= 1) ss += __shfl_xor(ss, off, 64);
      if (c % CPR == 0) sumsq[c / CPR] = ss;
    }
    __syncthreads();
    if (t < ROWS) sumsq[t] = (double)qknorm_rscale(sumsq[t], D, jb.norm.eps);
    __syncthreads();
    unsigned short* out = jb.norm_out != nullptr ? jb.norm_out + ((size_t)bh * Np + (size_t)blk * kBlock) * D : nullptr;
#pragma unroll
    for (int it = 0; it < NCH; it++) {
      const int c = t + 256 * it;
      const int row = c / CPR, ch = c % CPR;
      const float rs = (float)sumsq[row];
      const float* g = jb.norm.gamma + ch * 16;
      // (rows that do not exist are zero and stay zero; their factor 1 / sqrt(eps) is infinite for eps = 0)
      if (row < rows_here) {
#pragma unroll
        for (int e = 0; e < 16; e++) x[it][e] = qknorm_apply(x[it][e], rs, g[e]);
      }
      if (out != nullptr && row < nsub * kBlock) {
        v8us lo, hi;
#pragma unroll
        for (int e = 0; e < 8; e++) {
          lo[e] = float_to_bf16_bits(x[it][e]);        // exact: the values are bf16 already (zero in missing rows)
          hi[e] = float_to_bf16_bits(x[it][8 + e]);
        }
        unsigned short* o = out + (size_t)row * D + ch * 16;
        *(v8us*)o = lo;
        *(v8us*)(o + 8) = hi;
      }
    }
  }

  // x -= mu_s on the rows that exist
  auto subtract_mu = [&]() {
#pragma unroll
    for (int it = 0; it < NCH; it++) {
      const int row = (t + 256 * it) / CPR, ch = (t + 256 * it) % CPR;
      if (row < rows_here) {
#pragma unroll
        for (int e = 0; e < 16; e++) x[it][e] = x[it][e] - mu_s[ch * 16 + e];
      }
    }
  };

  // delta = rowsum(dO o O), FP32 (not part of the bit-exact contract)
  if (jb.O != nullptr) {
#pragma unroll
    for (int it = 0; it < NCH; it++) {
      const int c = t + 256 * it;
      const int row = c / CPR, ch = c % CPR;
      v8us lo = {0, 0, 0, 0, 0, 0, 0, 0}, hi = {0, 0, 0, 0, 0, 0, 0, 0};
      if (row < rows_here) {
        const unsigned short* p = jb.O + tile_off + (size_t)row * view.row_stride + ch * 16;
        lo = *(const v8us*)p;
        hi = *(const v8us*)(p + 8);
      }
      float acc = 0.f;
#pragma unroll
      for (int e = 0; e < 8; e++) {
        acc += x[it][e] * bf16_bits_to_float(lo[e]);
        acc += x[it][8 + e] * bf16_bits_to_float(hi[e]);
      }
#pragma unroll
      for (int off = 1; off < CPR; off <<= 1) acc += __shfl_xor(acc, off, 64);
      // stored negated: the backward starts the dP accumulators from -delta (dP - delta in one chain)
      if (ch == 0 && row < nsub * kBlock) jb.delta[(size_t)bh * Np + (size_t)blk * kBlock + row] = -acc;
    }
  }

  if (jb.lse != nullptr && t < nsub * kBlock) {
    const size_t row = (size_t)blk * kBlock + t;
    jb.nl2[(size_t)bh * Np + row] = t < rows_here ? -jb.lse[(size_t)bh * N + row] * 1.4426950408889634f : -INFINITY;
  }

  if (INLINE_MEAN && jb.mean_inline) {
    double acc[8];
    column_sums<D, MEAN == kMeanInlineNormed ? 4 : MEAN == kMeanInlineNormedBlock ? 1 : 0>(jb.src + view.row(bh, 0), view.row_stride, N, jb.norm, acc);
    // the rows of a wave meet in its first D / 8 lanes, the waves in colbuf
    double* red = (double*)colbuf;               // [wave][D]
    static_assert(4 * D * sizeof(double) <= sizeof(colbuf), "four waves' sums");
#pragma unroll
    for (int e = 0; e < 8; e++) {
#pragma unroll
      for (int off = D / 8; off < 64; off <<= 1) acc[e] += __shfl_xor(acc[e], off, 64);
      if ((t & 63) < D / 8) red[(t >> 6) * D + 8 * (t & 63) + e] = acc[e];
    }
    __syncthreads();
  }
  if ((INLINE_MEAN && jb.mean_inline) || jb.mean_part != nullptr) {
    // mu_K: the float64 sum of the head, divided by N, rounded once to FP32
    double* red = (double*)colbuf;
    const bool inline_mean = INLINE_MEAN && jb.mean_inline;
    if (!inline_mean) head_sums<D>(jb.mean_part + (size_t)bh * jb.nchunk * D, jb.nchunk, red);
    if (t < D) {
      double s = red[t];
#pragma unroll
      for (int g = 1; g < (INLINE_MEAN ? 4 : 256 / D); g++)
        if (inline_mean || g < 256 / D) s += red[g * D + t];
      const float m = (float)(s / (double)N);
      mu_s[t] = m;
      if (blk == 0) jb.mu_head_out[(size_t)bh * D + t] = m;
    }
    __syncthreads();
    subtract_mu();
  }

  if (jb.mu_head_out != nullptr && !(INLINE_MEAN && jb.mean_inline) && jb.mean_part == nullptr && blk == 0 && t < D)
    jb.mu_head_out[(size_t)bh * D + t] = 0.f;                               // no K-smoothing: the mean that was subtracted

  if (jb.mu_block_out != nullptr) {
    // block mean over the rows of the numerics block that exist: float64 column sums (exact for bf16 data; zeros where
    // a row does not exist), thread t < D taking channel t, 16 rows at a time through `colbuf`; one rounding
    double part = 0.0;
    for (int pass = 0; pass < ROWS / 16; pass++) {
      __syncthreads();
#pragma unroll
      for (int it = 0; it < NCH; it++) {
        const int c = t + 256 * it;
        const int row = c / CPR, ch = c % CPR;
        if (row / 16 == pass) {
#pragma unroll
          for (int e = 0; e < 16; e++) colbuf[(row % 16) * D + ch * 16 + e] = x[it][e];
        }
      }
      __syncthreads();
      if (t < D) {
        for (int r = 0; r < 16; r++) part += (double)colbuf[r * D + t];
      }
    }
    if (t < D) {
      const float m = (float)(part / (double)rows_here);
      mu_s[t] = m;
      for (int k = 0; k < nsub; k++) jb.mu_block_out[((size_t)bh * nblk + blk + k) * D + t] = m;
    }
    __syncthreads();
    subtract_mu();
  }

  // block absmax
  float a = 0.f;
#pragma unroll
  for (int it = 0; it < NCH; it++)
#pragma unroll
    for (int e = 0; e < 16; e++) a = fmaxf(a, fabsf(x[it][e]));
  a = wave_max_nonneg_f32(a);
  if ((t & 63) == 0) wmax[t >> 6] = a;
  __syncthreads();
  a = fmaxf(fmaxf(wmax[0], wmax[1]), fmaxf(wmax[2], wmax[3]));
  const bool nz = a > 0.f;
  const float s = nz ? a / 127.0f : 0.f;
  const float r = nz ? 127.0f / a : 0.f;
  if (t < nsub) jb.scale[(size_t)bh * nblk + blk + t] = s;

  const size_t frag_base = ((size_t)bh * (Np / 32) + (size_t)blk * 2) * (D / 32) * 1024;
#pragma unroll
  for (int it = 0; it < NCH; it++) {
    const int c = t + 256 * it;
    const int row = c / CPR, ch = c % CPR;
    const v4i packed = quantise_16(x[it], r);
    if (jb.outTF != nullptr) *(v4i*)(tile + row * D + ch * 16) = packed;
    if (jb.outF != nullptr && row < nsub * kBlock) {
      const int rb = row / 32, sstep = ch / 2, h = ch % 2;
      const int lane = (row % 32) + 32 * h;
      *(v4i*)(jb.outF + frag_base + ((size_t)(rb * (D / 32) + sstep) * 64 + lane) * 16) = packed;
    }
  }
  if (jb.outTF != nullptr) {
    __syncthreads();
#pragma unroll
    for (int it = 0; it < NTF; it++) {
      const int c = t + 256 * it;            // (rb, cb, lane)
      const int lane = c % 64, cb = (c / 64) % (D / 32), rb = c / (64 * (D / 32));
      if (rb >= 2 * nsub) break;             // (whole waves)
      const int col = 32 * cb + (lane % 32), h = lane / 32;
      v4i packed;
#pragma unroll
      for (int aa = 0; aa < 4; aa++) {
        unsigned u = 0;
#pragma unroll
        for (int b = 0; b < 4; b++) {
          const int row = 32 * rb + 8 * aa + 4 * h + b;
          u |= ((unsigned)(unsigned char)tile[row * D + col]) << (8 * b);
        }
        packed[aa] = (int)u;
      }
      *(v4i*)(jb.outTF + frag_base + ((size_t)(rb * (D / 32) + cb) * 64 + lane) * 16) = packed;
    }
  }
}

// ---- inspection: fragment layouts back to row-major -----------------------------
// One thread per 16-byte fragment chunk.  transposed = 0: F layout, 1: TF layout.
__global__ void export_fragments_kernel(const int8_t* __restrict__ frag, int8_t* __restrict__ out,
                                        size_t n_chunks, int N, int D, int transposed) {
  size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  if (i >= n_chunks) return;
  const int fpr = D / 32;                     // fragments per 32-row block
  const int lane = (int)(i % 64);
  const size_t f = i / 64;                    // global fragment index
  const int sc = (int)(f % fpr);
  const size_t rbg = f / fpr;                 // 32-row block over all heads (N % 32 == 0)
  const size_t head = rbg / (N / 32);
  const int rb = (int)(rbg % (N / 32));
  v4i v = *(const v4i*)(frag + i * 16);
  const int r = lane % 32, h = lane / 32;
  int8_t* obase = out + head * (size_t)N * D;
  if (!transposed) {
    *(v4i*)(obase + (size_t)(32 * rb + r) * D + 32 * sc + 16 * h) = v;
  } else {
#pragma unroll
    for (int aa = 0; aa < 4; aa++)
#pragma unroll
      for (int b = 0; b < 4; b++)
        obase[(size_t)(32 * rb + 8 * aa + 4 * h + b) * D + 32 * sc + r] = (int8_t)((v[aa] >> (8 * b)) & 0xff);
  }
}

// out = sign * in (sign = +-1: exact)
__global__ void copy_f32_kernel(const float* __restrict__ in, float* __restrict__ out, size_t n, float sign) {
  size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) out[i] = sign * in[i];
}

// ---- Q-smoothing: logit bias table -------------------------------------------------
// bias[bh][I][k] = sm_scale*log2(e) * mu_Q[I] . K_sm[k]  (the mu_Qi K_sm^T term of the
// Sec. 3 decomposition; the two mu_K terms are constant along a softmax row and dropped).
// FP32 from the unquantised K - mu_K.  Causal: blocks I < block(k) are never read (nor written).
template <int D>
__global__ void __launch_bounds__(256) qsmooth_bias_kernel(const unsigned short* __restrict__ K, RowView view,
                                                           const float* __restrict__ muK,
                                                           const float* __restrict__ muQ,
                                                           float* __restrict__ bias, int N, int Np, int nqblk,
                                                           int causal_shift, float scale_log2e) {
  // (N = rows of K as the caller holds it, Np = N rounded up to the block: keys that do not exist count as
  // zero rows; nqblk = Q blocks; causal_shift < 0: no mask, else Q block I sees key blocks <= I + causal_shift.)
  // One workgroup per (key block, head): a [Q blocks] x [64 keys] x [D channels] FP32 product on
  // the FP32 matrix instruction (32x32x2).  The smoothed keys go through LDS once (coalesced
  // reads); every wave keeps half of them as B operands in registers and takes 32 Q blocks at a
  // time as the A operand.  The contraction order is free, so lane (row, half) pairs channel
  // 8 v + 4 half + e with step (v, e): both operands then come from 16-byte reads.
  constexpr int LD = D + 4;                      // floats per LDS row (keeps rows 16-byte aligned)
  __shared__ __attribute__((aligned(16))) float ks[64 * LD];
  const int t = threadIdx.x;
  const int kblk = blockIdx.x, bh = blockIdx.y;
  const int nblk = Np / kBlock;
  const unsigned short* src = K + view.row(bh, (size_t)kblk * kBlock);
  const int rows_here = min(kBlock, N - kblk * kBlock);
  const float* mk = muK + (size_t)bh * D;
  {
    constexpr int NCH = 64 * D / 8 / 256;        // 16-byte chunks (8 channels) per thread
    v8us raw[NCH];
#pragma unroll
    for (int u = 0; u < NCH; u++) {
      raw[u] = v8us{0, 0, 0, 0, 0, 0, 0, 0};
      const int ch = t + 256 * u;
      if (ch / (D / 8) < rows_here) raw[u] = *(const v8us*)(src + (size_t)(ch / (D / 8)) * view.row_stride + 8 * (ch % (D / 8)));
    }
#pragma unroll
    for (int u = 0; u < NCH; u++) {
      const int ch = t + 256 * u, row = ch / (D / 8), c0 = 8 * (ch % (D / 8));
      const bool there = row < rows_here;
      const v4f m0 = *(const v4f*)(mk + c0), m1 = *(const v4f*)(mk + c0 + 4);
      v4f f0, f1;
#pragma unroll
      for (int e = 0; e < 4; e++) {
        f0[e] = there ? bf16_bits_to_float(raw[u][e]) - m0[e] : 0.f;
        f1[e] = there ? bf16_bits_to_float(raw[u][4 + e]) - m1[e] : 0.f;
      }
      *(v4f*)(ks + row * LD + c0) = f0;
      *(v4f*)(ks + row * LD + c0 + 4) = f1;
    }
  }
  __syncthreads();
  const int lane = t & 63, r = lane & 31, half = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  // wave = (Q-block tile parity, key half): each wave keeps one half of the keys as B operands
  const int kt = wave & 1;
  v4f kb[D / 8];                                 // B operands: key 32 kt + r
#pragma unroll
  for (int v = 0; v < D / 8; v++) kb[v] = *(const v4f*)(ks + (32 * kt + r) * LD + 8 * v + 4 * half);
  const int first = causal_shift >= 0 ? max(kblk - causal_shift, 0) : 0;   // Q blocks that cannot see the key block are never read
  for (int it = first / 32 + (wave >> 1); 32 * it < nqblk; it += 2) {
    const int I = min(32 * it + r, nqblk - 1);   // rows past the end repeat the last one (not stored)
    const float* mq = muQ + ((size_t)bh * nqblk + I) * D + 4 * half;
    v16f acc[2];                                 // two chains over alternate steps, summed at the end
#pragma unroll
    for (int c = 0; c < 2; c++)
#pragma unroll
      for (int e = 0; e < 16; e++) acc[c][e] = 0.f;
#pragma unroll
    for (int v = 0; v < D / 8; v++) {
      const v4f a4 = *(const v4f*)(mq + 8 * v);
#pragma unroll
      for (int e = 0; e < 4; e++)
        acc[e & 1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a4[e], kb[v][e], acc[e & 1], 0, 0, 0);
    }
    // accumulator register e of lane (r, half): Q block 32 it + 8 (e / 4) + 4 half + e % 4, key 32 kt + r
#pragma unroll
    for (int e = 0; e < 16; e++) {
      const int Io = 32 * it + 8 * (e >> 2) + 4 * half + (e & 3);
      if (Io >= first && Io < nqblk)
        bias[((size_t)bh * nqblk + Io) * Np + (size_t)kblk * kBlock + 32 * kt + r] = (acc[0][e] + acc[1][e]) * scale_log2e;
    }
  }
}

// The same table for at most 16 Q blocks, where the kernel above has no Q blocks for two of its waves and half a tile of rows that do
// not exist for the others: wave w forms 16 Q blocks x keys 16 w .. with 16x16x4 products, both operands straight from the tensors,
// without LDS or a barrier.  Step (v, p) contracts channels 8 v + p + 0, 4, 2, 6 in the four lanes of a row, which is the order in
// which two steps of the kernel above do: the same bits, so that no logit falls to the other side of a rounding.  The four lanes of
// a row read whole 16-byte pieces.  Bound by latency, as the kernel above is there: 0.5 to 0.9 us less of a call (the forward of 8
// heads of N = 512 23.2 -> 22.6, of 40 heads of 41 14.6 -> 13.7; see use_bias_short for where it is chosen).
template <int D>
__global__ void __launch_bounds__(256) qsmooth_bias_short_kernel(const unsigned short* __restrict__ K, RowView view,
                                                                 const float* __restrict__ muK, const float* __restrict__ muQ,
                                                                 float* __restrict__ bias, int N, int Np, int nqblk,
                                                                 int causal_shift, float scale_log2e) {
  const int kblk = blockIdx.x, bh = blockIdx.y;
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int c0 = 4 * (g & 1) + 2 * (g >> 1);     // first channel of the lane's in every eight
  const int key = kblk * kBlock + 16 * __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);     // first of the wave
  const unsigned short* src = K + view.row(bh, min(key + r, N - 1)) + c0;
  const float* mk = muK + (size_t)bh * D + c0;
  const float* mq = muQ + ((size_t)bh * nqblk + min(r, nqblk - 1)) * D + c0;                 // Q blocks past the end repeat the last one (not stored)
  v4f acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};                                 // two chains over alternate channels, summed at the end
#pragma unroll
  for (int v = 0; v < D / 8; v++) {
    const unsigned raw = *(const unsigned*)(src + 8 * v);
    const v2f m = *(const v2f*)(mk + 8 * v), q = *(const v2f*)(mq + 8 * v);
#pragma unroll
    for (int p = 0; p < 2; p++) {
      const float k = key + r < N ? bf16_bits_to_float((unsigned short)(raw >> (16 * p))) - m[p] : 0.f;      // keys that do not exist count as zero rows
      acc[p] = __builtin_amdgcn_mfma_f32_16x16x4f32(k, q[p], acc[p], 0, 0, 0);
    }
  }
  // register e of lane (r, g): key 4 g + e of the wave, Q block r
  if (r < nqblk && (causal_shift < 0 || kblk <= r + causal_shift)) {
    v4f o;
#pragma unroll
    for (int e = 0; e < 4; e++) o[e] = (acc[0][e] + acc[1][e]) * scale_log2e;
    *(v4f*)(bias + ((size_t)bh * nqblk + r) * Np + key + 4 * g) = o;
  }
}

// ---- inspection: the psi(dS) tiles the backward left in its scratch, as a row-major [Np, Np] matrix ----
// Tile (i, j) holds four 1 KiB fragments (32-query block qb, 32-key block kb): lane (key, half), byte
// 4 a + b = psi(dS)[64 i + 32 qb + 8 a + 4 half + b][64 j + 32 kb + key] (a quantised accumulator quadrant
// as the backward kernel holds it).  Tiles above the causal diagonal
// were never written: they are returned as zeros.  One thread per 16 bytes.
__global__ void export_ds_kernel(const int8_t* __restrict__ tiles, const float* __restrict__ scales,
                                 int8_t* __restrict__ ds_out, float* __restrict__ scale_out, int nqblk, int Np,
                                 int pitch, int causal_shift) {
  // [nqblk * 64, Np] out; causal_shift < 0: no mask, else tile (i, j) exists iff j <= i + causal_shift
  const int nblk = Np / kBlock;
  const size_t c = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  if (c >= (size_t)nqblk * nblk * 256) return;
  const int tile = (int)(c / 256), i = tile / nblk, j = tile % nblk;
  const int frag = (int)(c % 256) / 64, lane = (int)(c % 64);
  const bool there = causal_shift < 0 || j <= i + causal_shift;
  v4i v = {0, 0, 0, 0};
  if (there) v = *(const v4i*)(tiles + ((size_t)i * pitch + j) * 4096 + (c % 256) * 16);   // `pitch` tiles per Q-block row
  // fragment (qb, kb), lane (key, h), byte 4 a + b = psi(dS)[32 qb + 8 a + 4 h + b][32 kb + key]
  const int qrow0 = 64 * i + 32 * (frag >> 1) + 4 * (lane >> 5), key = 64 * j + 32 * (frag & 1) + (lane & 31);
  if (ds_out != nullptr) {
#pragma unroll
    for (int a = 0; a < 4; a++)
#pragma unroll
      for (int b = 0; b < 4; b++) ds_out[(size_t)(qrow0 + 8 * a + b) * Np + key] = (int8_t)((v[a] >> (8 * b)) & 0xff);
  }
  if (scale_out != nullptr && c % 256 == 0) scale_out[tile] = there ? scales[(size_t)i * pitch + j] : 0.f;
}

}  // namespace sage
