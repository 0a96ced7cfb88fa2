// Fused INT8 attention forward (paper Algorithm 1) for gfx950.
//
// One wave owns 32 queries; a workgroup of NW waves owns 32*NW consecutive queries of
// one head and walks the KV blocks (64 keys each).  K^ and V^ fragments are copied
// global -> LDS asynchronously into a ring of four tile buffers, one barrier per tile.
//
// The logits are formed TRANSPOSED, S^T = K^ Q^^T (keys x queries), with the 32x32x32
// INT8 MFMA: an accumulator lane then holds one query (column) and 16 keys (rows) per
// 32-key block, so that
//   - the row max / row sum of the softmax are in-lane reductions plus one exchange
//     between the two half-waves,
//   - the per-token quantised P^ (Algorithm 1 line 9), packed four codes to a register,
//     is already the B operand of O^T = V^^T P^^T (the TF layout of V^ orders its keys
//     the way the accumulator holds them), with no trip through LDS.
//
// Software pipeline inside a wave: the MFMAs of S_{j+1} are issued before the softmax of
// tile j, and the MFMAs of one 32-channel block of P^V^ before the FP32 update of the
// previous block, so that the matrix pipe works underneath the vector work of the same wave.
//
// Per-token quantisation: P~/s_P with s_P = exp(rowmax(S_ij) - m_ij)/127 equals
// 127 * exp(S_ij - rowmax(S_ij)), which does not depend on the running max.  The kernel
// evaluates that form (never 0/0) and keeps the running reference m only for the FP32
// accumulators: O += beta * s_V * (P^ V^), l += beta * sum(127 p), beta = exp(rowmax - m).
// m is raised only when a tile's row max exceeds it by more than kTau (in log2 units); the
// result is unchanged because O/l and m + log l do not depend on the reference chosen.
//
// INT32 -> FP32 without a conversion instruction: the P^V^ accumulators start from the bit
// pattern B0 of the float C0 = 1/(2 pi) (an inline constant of the ISA, see mfma_from_bias).  B0's mantissa leaves more than 2^20
// codes to either end of its binade, so for every possible sum |a| <= 64 * 127 * 127 the bits B0 + a read as the float C0 + a * 2^-26
// exactly.  The FP32 accumulators take w * 2^26 * (C0 + a * 2^-26) with ONE fused multiply-add
// per value and so carry the bias C0 * 2^26 * sum(w), the same for every channel of a query;
// it is subtracted every kBiasPeriod tiles and at the end.  Between corrections the bias stays
// below about 2^26 times the weight of a tile, so each addition still resolves a * w to about
// one part in 10^4 of a typical tile's contribution.  Measured at N = 8192 against the CPU oracle:
// relative L1 of O 2.5e-4 (6e-5 when the bias is subtracted after every tile, 4e-4 with a period
// of 16), an order of magnitude below the rounding of the bf16 output and the 1e-2 tolerance.
// The logits' accumulators use the same start where the tile scales allow it (SBIAS in fwd_tile;
// |s| <= 128 * 127 * 127 still fits the binade): O then sits 5e-4 from the oracle, L 4e-5.
#pragma once

#include <type_traits>

#include "common.h"

namespace sage {

struct FwdArgs {
  const int8_t* QF;     // F layout
  const int8_t* KF;     // F layout
  const int8_t* VT;     // TF layout
  const float* sQ;      // [BH, N/64]
  const float* sK;
  const float* sV;
  const float* bias;    // Q-smoothing: [BH, N/64, N] = sm_scale*log2e * mu_Qi . K_sm[k], else nullptr
  unsigned short* O;    // bf16, rows addressed through `oview` (dense [BH, N, D] or the caller's token-major tensor)
  RowView oview;
  float* LSE;           // [BH, nq_valid]
  int BH, N;            // N = rows of the K-like workspace tensors (N_kv rounded up to a multiple of 64)
  int nvalid;           // keys >= nvalid do not exist (nvalid = N unless N_kv is not a multiple of 64)
  int Nq;               // rows of the Q-like workspace tensors (N_q rounded up to a multiple of 64)
  int nq_valid;         // query rows >= nq_valid do not exist
  int shift;            // causal: query i sees keys k <= i + shift (N_kv - N_q, a multiple of 64)
  int n_qtiles;         // workgroups per head
  int head_set;         // heads per XCD whose work items are interleaved (see work_item)
  int fold_end;         // order of the first workgroups (see folded)
  float scale_log2e;    // sm_scale * log2(e)
};

constexpr float kTau = 8.0f;
constexpr float kLog2_127 = 6.98868468677216585f;
constexpr float kLn2 = 0.69314718055994531f;
constexpr int kBiasPeriod = 8;                // tiles between two subtractions of the accumulated bias

// Keeps the computation of `v` where it is written: without a use at this point the compiler
// sinks the vector work of a chunk past the scheduling barriers into the next basic block.
__device__ __forceinline__ void pin(float& v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ void pin_i(int& v) { asm volatile("" : "+v"(v)); }

// S^T accumulators of one 64-key tile (two 32-key blocks), interleaved so that consecutive
// MFMAs are independent.
template <int D, bool SBIAS>
__device__ __forceinline__ void fwd_s_mfma(const int8_t* __restrict__ Kt, const v4i (&qf)[D / 32], v16i (&sacc)[2],
                                           const int lane) {
  constexpr int KS = D / 32;
#pragma unroll
  for (int kb = 0; kb < 2; kb++)
#pragma unroll
    for (int r = 0; r < 16; r++) sacc[kb][r] = SBIAS ? kBiasBits : 0;
#pragma unroll
  for (int s = 0; s < KS; s++) {
#pragma unroll
    for (int kb = 0; kb < 2; kb++) {
      const v4i a = *(const v4i*)(Kt + (kb * KS + s) * 1024 + lane * 16);
      sacc[kb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, qf[s], sacc[kb], 0, 0, 0);
    }
  }
}

// One KV tile for one wave: (optionally) the logits of the NEXT tile on the matrix pipe, the
// softmax and per-token quantisation of THIS tile (`sacc`), then O^T += V^^T P^^T.
// MASK = the tile straddles the causal diagonal for this wave.
//
// The instruction stream is laid out by hand in chunks separated by scheduling barriers: each
// chunk pairs one MFMA (and the LDS read of an operand two MFMAs ahead) with the vector work of
// four logits or of sixteen output values, so that the matrix pipe and the LDS latency hide
// under the vector instructions of the same wave.  `copy(k)` issues the k-th of this wave's global -> LDS
// copies for a coming tile, one in every second slot: alone a wave issues such a copy in 12 cycles, but the CU takes
// one in 16, and four copies of each of its eight waves in one place hold every wave for about 200 of a tile's 3000 cycles.
//
// CARRY = the row max of this tile's logits was taken under the last tile's output update and comes in `carried` (over the two lane
// halves); that of the next tile, unmasked, goes out there.  It takes a chain of some 20 dependent instructions out of the
// tile's head (2 to 3 % of the kernel).  The exponents of a slot are formed in the slot before (another 2 to 3 %).
//
// KV128 = numerics blocks of 128 keys: the per-token quantiser of P~ (Algorithm 1 line 9) then takes its row
// max over both 64-key tiles of the block.  `pair` carries the other tile's row max in (INT_MIN / -inf if
// the other tile has no visible key) and this tile's own row max out.
struct PairMax {
  int i;      // integer domain (no Q-smoothing: both tiles of a block share the scale c)
  float f;    // log2 domain (Q-smoothing)
};
template <int D, bool QSMOOTH, bool MASK, bool NEXT, bool SBIAS, bool KV128 = false, bool CARRY = false, class Copy>
__device__ __forceinline__ void fwd_tile(const Copy& copy, const int8_t* __restrict__ Knext, const int8_t* __restrict__ Vt,
                                         const v4i (&qf)[D / 32], v16i (&sacc)[2], v16i (&snext)[2],
                                         float (&oacc)[D / 32][16], float& w_bias, float& m_ref, float (&l_part)[2],
                                         const float c, const float sv, const float* __restrict__ bias_row,
                                         const int k0, const int q, const int lane, const int h,
                                         PairMax* pair = nullptr, int* carried = nullptr) {
  constexpr int KS = D / 32;
  constexpr int NSM = 2 * KS;    // MFMAs of the next tile's logits; MFMA m = (k-step m / 2, key block m % 2)
  const int8_t* kl = Knext + lane * 16;
  const int8_t* vl = Vt + lane * 16;
  auto k_frag = [&](int m) { return *(const v4i*)(kl + ((m & 1) * KS + (m >> 1)) * 1024); };
  auto v_frag = [&](int m) { return *(const v4i*)(vl + m * 1024); };   // m = kb * KS + cb

  v4i ka[3];
  if constexpr (NEXT) {
    ka[0] = k_frag(0);
    ka[1] = k_frag(1);
  }

  float x[2][16];
  float mloc;   // row max of the tile in the log2 domain
  float bmax_f = 0.f;   // SBIAS: the row max as the float its bits spell
  if constexpr (!QSMOOTH) {
    // the scale is one positive scalar per tile, so the row max can be taken on the integers
    int mrow;
    if constexpr (CARRY) {
      mrow = *carried;
    } else {
      int mi[2] = {INT_MIN, INT_MIN};
#pragma unroll
      for (int kb = 0; kb < 2; kb++)
#pragma unroll
        for (int r = 0; r < 16; r++) {
          int v = sacc[kb][r];
          if constexpr (MASK) {
            const int key = k0 + 32 * kb + 8 * (r >> 2) + 4 * h + (r & 3);
            v = key > q ? INT_MIN : v;
            sacc[kb][r] = v;
          }
          mi[kb] = max(mi[kb], v);
        }
    // (with SBIAS the accumulators hold B0 + s: the same order, and B0 + s never is INT_MIN)
      mrow = half_swap_max_i32(max(mi[0], mi[1]));
    }
    if constexpr (KV128) {
      const int own = mrow;
      mrow = max(mrow, pair->i);
      pair->i = own;
    }
    mloc = (float)(mrow - (SBIAS ? kBiasBits : 0)) * c;
    if constexpr (SBIAS) bmax_f = __int_as_float(mrow);
  } else {
    float mf = -INFINITY;
#pragma unroll
    for (int kb = 0; kb < 2; kb++)
#pragma unroll
      for (int aa = 0; aa < 4; aa++) {
        const int key = k0 + 32 * kb + 8 * aa + 4 * h;
        const v4f b4 = *(const v4f*)(bias_row + (key - k0));   // the tile's 64 biases, staged in LDS
#pragma unroll
        for (int b = 0; b < 4; b++) {
          float v = __builtin_fmaf((float)sacc[kb][4 * aa + b], c, b4[b]);
          if constexpr (MASK) v = (key + b) > q ? -INFINITY : v;
          x[kb][4 * aa + b] = v;
          mf = fmaxf(mf, v);
        }
      }
    mloc = half_swap_max_f32(mf);
    if constexpr (KV128) {
      const float own = mloc;
      mloc = fmaxf(mloc, pair->f);
      pair->f = own;
    }
  }
  // ---- online softmax reference (rarely raised) ----
  if (__builtin_amdgcn_ballot_w64(mloc > m_ref + kTau) != 0) {
    const float m_new = fmaxf(m_ref, mloc);
    const float alpha = __builtin_amdgcn_exp2f(m_ref - m_new);   // 0 on the first tile
    l_part[0] *= alpha;
    l_part[1] *= alpha;
    w_bias *= alpha;
#pragma unroll
    for (int cb = 0; cb < KS; cb++)
#pragma unroll
      for (int r = 0; r < 16; r++) oacc[cb][r] *= alpha;
    m_ref = m_new;
  }
  const float beta = __builtin_amdgcn_exp2f(mloc - m_ref);
  // SBIAS: the logits' accumulators started from the bits of C0, so they read as the floats
  // C0 + s * 2^-26 and x = s * c + off becomes one FMA on those floats, without a conversion; the
  // offset is formed from the row max taken the same way, so the largest logit of the row still
  // lands on log2(127) up to the rounding of the product C0 * 2^26 * c (the caller admits only
  // scales c for which that is far below the half code that would carry 127 to 128).
  const float c_eff = SBIAS ? c * kTwo26 : c;
  const float off = SBIAS ? __builtin_fmaf(-bmax_f, c_eff, kLog2_127) : kLog2_127 - mloc;
  // exponents of a group of four logits (group g: key block g / 4, registers 4 (g % 4) ..), formed one slot ahead of their exp2
  float xn[4];
  auto form_x = [&](int g) __attribute__((always_inline)) {
    const int kb = g >> 2, aa = g & 3;
#pragma unroll
    for (int b = 0; b < 4; b++) {
      float xv;
      if constexpr (!QSMOOTH) {
        if constexpr (SBIAS) xv = __builtin_fmaf(__int_as_float(sacc[kb][4 * aa + b]), c_eff, off);
        else xv = __builtin_fmaf((float)sacc[kb][4 * aa + b], c, off);
        if constexpr (MASK) xv = sacc[kb][4 * aa + b] == INT_MIN ? -INFINITY : xv;
      } else {
        xv = x[kb][4 * aa + b] + off;
      }
      xn[b] = xv;
    }
  };
  form_x(0);
  __builtin_amdgcn_sched_barrier(0);

  // ---- slots 0..7: P^ = rne(127 exp(S - rowmax)) for four logits each, packed as the B operand;
  //      row sum of 127 p.  Matrix work issued underneath: MFMA m of the next tile's logits in
  //      slot m; the first half of O^T += V^^T P^^T (key block 0, channel block cb) in slot 4 + cb.
  // ---- slots 8..: the second half (key block 1) in slot 8 + cb, and the FP32 update of channel
  //      block cb in slots 10 + 2 cb and 11 + 2 cb.  V^ fragments are read two slots ahead. ----
  v4i pf[2];
  v4i va[4];
  v16i t[KS];
  float psum[4] = {0.f, 0.f, 0.f, 0.f};
  float w = 0.f;
  int nmax[2] = {INT_MIN, INT_MIN};
  constexpr int NSLOT = 10 + 2 * KS;
  static_assert(NSLOT >= 14, "the next tile's row max takes slots 8 to 13");
  auto pv_slot = [&](int m) { return m < KS ? 4 + m : 8 + (m - KS); };   // slot of P^V^ MFMA m = (kb, cb)
#pragma unroll
  for (int sl = 0; sl < NSLOT; sl++) {
    // The softmax slots carry the long dependency chains (max, exp2, pack); a wave in them gets issue
    // priority over its SIMD neighbour, which is mostly in the matrix-heavy second half (measured: 5-7 %).
    if (sl == 0) __builtin_amdgcn_s_setprio(1);
    if (sl == 8) __builtin_amdgcn_s_setprio(0);
    if (sl & 1) copy(sl >> 1);
    // LDS reads: V^ fragment of the MFMA two slots ahead
#pragma unroll
    for (int m = 0; m < 2 * KS; m++)
      if (pv_slot(m) == sl + 2) va[m & 3] = v_frag(m);
    // matrix work of this slot
    if constexpr (NEXT) {
      if (sl < NSM) {
        if (sl + 2 < NSM) ka[(sl + 2) % 3] = k_frag(sl + 2);
        if (sl < 2) {
          v16i z;
#pragma unroll
          for (int r = 0; r < 16; r++) z[r] = 0;
          snext[sl & 1] = SBIAS ? mfma_from_bias(ka[sl % 3], qf[sl >> 1]) : __builtin_amdgcn_mfma_i32_32x32x32_i8(ka[sl % 3], qf[sl >> 1], z, 0, 0, 0);
        } else {
          snext[sl & 1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(ka[sl % 3], qf[sl >> 1], snext[sl & 1], 0, 0, 0);
        }
      }
    }
#pragma unroll
    for (int m = 0; m < 2 * KS; m++)
      if (pv_slot(m) == sl) {
        if (m < KS) {
          t[m] = mfma_from_bias(va[m & 3], pf[0]);
        }
        else t[m - KS] = __builtin_amdgcn_mfma_i32_32x32x32_i8(va[m & 3], pf[1], t[m - KS], 0, 0, 0);
      }
    // vector work of this slot
    if (sl < 8) {
      const int kb = sl >> 2, aa = sl & 3;
      unsigned u = 0;
      float e[4];
#pragma unroll
      for (int b = 0; b < 4; b++) e[b] = __builtin_amdgcn_exp2f(xn[b]);
      __builtin_amdgcn_sched_barrier(0);
      if (sl < 7) form_x(sl + 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int b = 0; b < 4; b++) {
        psum[b] = aa == 0 ? e[b] : psum[b] + e[b];
        pin(psum[b]);
        u = __builtin_amdgcn_cvt_pk_u8_f32(e[b], b, u);
      }
      pf[kb][aa] = (int)u;
      if (aa == 3) {
        // (one sum per key block, which meet at the end: sage_fwd_pair_kernel has them in two waves)
        l_part[kb] = __builtin_fmaf(beta, (psum[0] + psum[1]) + (psum[2] + psum[3]), l_part[kb]);
        pin(l_part[kb]);
      }
    }
    if constexpr (NEXT && CARRY) {
      if (sl == 8) nmax[0] = max(max(snext[0][0], snext[0][1]), snext[0][2]);
      if (sl == 9) {
#pragma unroll
        for (int r = 3; r < 15; r += 2) nmax[0] = max(max(snext[0][r], snext[0][r + 1]), nmax[0]);
        pin_i(nmax[0]);
      }
      if (sl >= 10 && sl < 13) {
        if (sl == 10) nmax[1] = max(snext[1][0], snext[0][15]);
#pragma unroll
        for (int r = 1; r < 15; r += 2)
          if ((r < 5 ? 10 : r < 11 ? 11 : 12) == sl) nmax[1] = max(max(snext[1][r], snext[1][r + 1]), nmax[1]);
        if (sl == 12) nmax[0] = max(max(snext[1][15], nmax[0]), nmax[1]);
        pin_i(nmax[1]);
        pin_i(nmax[0]);
      }
      if (sl == 13) {
        *carried = half_swap_max_i32(nmax[0]);
        pin_i(*carried);
      }
    }
    if (sl == 8) {
      w = beta * sv * kTwo26;
      w_bias += w;
      pin(w);
      pin(w_bias);
    } else if (sl >= 10) {
      const int cb = (sl - 10) >> 1, half = (sl - 10) & 1;
#pragma unroll
      for (int r = 8 * half; r < 8 * half + 8; r++) {
        oacc[cb][r] = __builtin_fmaf(__int_as_float(t[cb][r]), w, oacc[cb][r]);
        pin(oacc[cb][r]);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

// Row max of one tile's logits `s` over the keys a lane's query sees (key <= qlim), as fwd_tile forms it:
// the integer max (no Q-smoothing) or the max of s * c + bias in the log2 domain.
template <bool QSMOOTH, bool MASK>
__device__ __forceinline__ PairMax tile_row_max(const v16i (&s)[2], const float c, const float* __restrict__ bias_row,
                                                const int k0, const int qlim, const int h) {
  PairMax m{INT_MIN, -INFINITY};
#pragma unroll
  for (int kb = 0; kb < 2; kb++)
#pragma unroll
    for (int aa = 0; aa < 4; aa++) {
      const int key = k0 + 32 * kb + 8 * aa + 4 * h;
      v4f b4 = {0.f, 0.f, 0.f, 0.f};
      if constexpr (QSMOOTH) b4 = *(const v4f*)(bias_row + (key - k0));
#pragma unroll
      for (int b = 0; b < 4; b++) {
        const bool hidden = MASK && (key + b) > qlim;
        if constexpr (QSMOOTH) {
          const float v = __builtin_fmaf((float)s[kb][4 * aa + b], c, b4[b]);
          m.f = fmaxf(m.f, hidden ? -INFINITY : v);
        } else {
          m.i = max(m.i, hidden ? INT_MIN : s[kb][4 * aa + b]);
        }
      }
    }
  if constexpr (QSMOOTH) m.f = half_swap_max_f32(m.f);
  else m.i = half_swap_max_i32(m.i);
  return m;
}

template <int D, bool CAUSAL, bool QSMOOTH, int NW, bool KV128 = false>
__global__ void __launch_bounds__(64 * NW, D == 64 ? 3 : 2) sage_fwd_kernel(FwdArgs args) {
  constexpr int KS = D / 32;                 // k-steps of Q K^T; also channel blocks of O
  constexpr int TILE_BYTES = 64 * D;         // one K^ or V^ tile of 64 keys
  constexpr int PAIR = 2 * TILE_BYTES;       // K^ tile | V^ tile
  constexpr int NFRAG = PAIR / 1024;         // 1 KiB fragments per pair
  constexpr int QT = 32 * NW;                // queries per workgroup

  // Q-smoothing: the 64 logit biases of each wave's Q block and the tile's keys travel with the tile too
  constexpr int BIAS_OFF = PAIR;
  constexpr int SLOT = BIAS_OFF + (QSMOOTH ? NW * 256 : 0);
  __shared__ __attribute__((aligned(16))) int8_t lds[4][SLOT];   // K^ | V^ | per-wave bias row

  // workgroup -> (head, query tile): a head's tiles share one XCD's L2; heaviest (last) query
  // tiles first under the causal mask, over sets of heads (see work_item)
  const WorkItem wi = work_item(folded(blockIdx.x, args.fold_end), args.n_qtiles, args.head_set);
  const int bh = wi.head;
  const int qt = args.n_qtiles - 1 - wi.item;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ql = lane & 31, h = lane >> 5;
  const int N = args.N;
  // First query of this wave.  The last workgroup of an odd number of Q blocks has two waves without queries: they take part in
  // the copies and the barriers, form nothing and store nothing (q0: rows that exist, for the loads of the prologue).  (Workgroups of 64
  // queries served such calls before: half the waves to share a staged tile, and 6 heads of N = 22028, blocks of 128, took 998 us
  // where N = 22016 took 677; now 705.)
  const int q0w = qt * QT + 32 * wave;
  const bool has_rows = q0w < args.Nq;
  const int q0 = has_rows ? q0w : args.Nq - 32;
  const int q = q0w + ql;
  // last visible key of this lane's query: under the causal mask the query's own position among the
  // keys (a query row that does not exist may see keys that do not exist: it is dropped anyway), else
  // the last key
  const int qlim = CAUSAL ? q + args.shift : args.nvalid - 1;
  const int nblk = N / kBlock;               // KV blocks
  const int nqblk = args.Nq / kBlock;        // Q blocks

  const int8_t* KFh = args.KF + (size_t)bh * N * D;
  const int8_t* VTh = args.VT + (size_t)bh * N * D;
  const float* sKh = args.sK + (size_t)bh * nblk;
  const float* sVh = args.sV + (size_t)bh * nblk;

  // Q^ fragments stay in registers for the whole loop
  v4i qf[KS];
  {
    const int8_t* p = args.QF + (size_t)bh * args.Nq * D + (size_t)(q0 / 32) * KS * 1024 + lane * 16;
#pragma unroll
    for (int s = 0; s < KS; s++) qf[s] = *(const v4i*)(p + s * 1024);
  }
  const float cq = args.sQ[(size_t)bh * nqblk + q0 / kBlock] * args.scale_log2e;
  const float* bias_row = QSMOOTH ? args.bias + ((size_t)bh * nqblk + q0 / kBlock) * N : nullptr;

  const int n_tiles = CAUSAL ? min((qt * QT + QT + args.shift) / kBlock, nblk) : nblk;   // barrier count, uniform in the workgroup
  const int last = CAUSAL ? (q0 + 31 + args.shift) / kBlock : nblk - 1;       // this wave's last tile (masked if causal)

  float oacc[KS][16];
#pragma unroll
  for (int cb = 0; cb < KS; cb++)
#pragma unroll
    for (int r = 0; r < 16; r++) oacc[cb][r] = 0.f;
  float w_bias = 0.f;        // sum of the tile weights since the last bias subtraction (see the header)
  float m_ref = -INFINITY;   // log2 domain
  float l_part[2] = {0.f, 0.f};   // this lane's share of sum(127 p) relative to m_ref, per 32-key block of the tiles

  // Asynchronous copy of tile j (K^ fragments, then V^ fragments) into a ring slot; the
  // 1 KiB fragments are dealt round-robin to the waves.
  constexpr int CPW = NFRAG / NW + (QSMOOTH ? 1 : 0);   // copies per wave and tile
  unsigned lane16 = lane * 16;
  static_assert(NFRAG % NW == 0, "every wave must issue the same number of copies");
  static_assert(NFRAG / 2 % NW == 0, "a copy is of K^ for every wave, or of V^");
  auto copy_piece = [&](int j, int8_t* dst, int k) __attribute__((always_inline)) {
    const int o = wave + NW * k;             // wave-uniform
    if (k < NFRAG / 2 / NW) copy_16(uniform(KFh + (size_t)j * TILE_BYTES + o * 1024) + lane16, dst + o * 1024);
    else if (k < NFRAG / NW) copy_16(uniform(VTh + (size_t)j * TILE_BYTES + (o - NFRAG / 2) * 1024) + lane16, dst + o * 1024);
    else if (QSMOOTH && k == NFRAG / NW) copy_4(uniform(bias_row + j * kBlock) + (lane16 >> 2), dst + BIAS_OFF + wave * 256);
  };
  auto stage_load = [&](int j, int8_t* dst) {
#pragma unroll
    for (int k = 0; k < CPW; k++) copy_piece(j, dst, k);
  };

  int8_t* cur = &lds[0][0];
  int8_t* nxt = &lds[1][0];
  int8_t* nx2 = &lds[2][0];
  int8_t* nx3 = &lds[3][0];
  stage_load(0, cur);
  if (n_tiles > 1) stage_load(1, nxt);
  if (n_tiles > 2) stage_load(2, nx2);
  barrier_all_memory();


  // Iteration j: tile j + 3 starts to load into the slot that tile j - 1 occupied (every wave is
  // past the barrier that ended iteration j - 1, so nobody reads it any more); this wave forms
  // S_{j+1} from slot `nxt` and finishes tile j with V^ from slot `cur`; before the barrier at
  // the end it waits for the copies of tile j + 2 (issued one iteration earlier), while its copies
  // of tile j + 3 stay in flight (from an unmasked iteration past the last tile that one again, never read: without a branch around
  // each copy the tile is one basic block, 1 to 3 % of the kernel).  The block scales come one tile ahead through the scalar cache, so the
  // loop has no register-returning vector loads whose waits would also drain the copies.  Every wave of
  // the workgroup runs n_tiles iterations (the barriers must match): its unmasked tiles, its last
  // tile, then iterations that only keep the ring moving.
  auto end_iter = [&](const bool issued) __attribute__((always_inline)) {
    if (issued) {
      __builtin_amdgcn_s_waitcnt(vmcnt_only(CPW));   // vmcnt: all but this iteration's copies
      barrier_lds_only();
    } else {
      barrier_all_memory();
    }
    int8_t* t = cur;
    cur = nxt;
    nxt = nx2;
    nx2 = nx3;
    nx3 = t;
  };
  // An iteration after the wave's last tile.  From that tile on a copy is issued only where there is a tile, so the last wait of the
  // workgroup is for everything and short calls copy no tile twice (numerics blocks of 128 keys also lose the registers that the clamped
  // addresses held: 116 bytes of scratch -> 0).  With this and waves without queries that form nothing, forward calls in us: 2048 heads of
  // N = 192, d = 64, 92.9 -> 90.3, 1100 of N = 40, d = 128, 31.7 -> 31.0, 4096 of N = 64 112.6 -> 111.2, 600 of N = 128 with blocks
  // of 128 keys, d = 64, 27.6 -> 26.3.
  auto keep_ring_moving = [&](const int j) {
    const bool issue = j + 3 < n_tiles;
    if (issue) stage_load(j + 3, nx3);
    end_iter(issue);
  };
  if (!has_rows) {
    for (int j = 0; j < n_tiles; j++) keep_ring_moving(j);
    return;
  }
  // subtracts the bias that the output accumulators carry (see the header)
  auto unbias = [&]() {
    const float corr = kBiasC0 * w_bias;
#pragma unroll
    for (int cb = 0; cb < KS; cb++)
#pragma unroll
      for (int r = 0; r < 16; r++) oacc[cb][r] -= corr;
    w_bias = 0.f;
  };
  // The logits' accumulators can start from the bits of C0 as well (SBIAS, see fwd_tile), which
  // saves the INT32 -> FP32 conversion of every logit; that needs C0 * 2^26 * c, about 1e7 c, to
  // stay small against the half code between 127 and 128 in the log2 domain, so the wave takes
  // that path only if its largest tile scale c is below 1e-3 (QK-normed inputs sit near 1e-4).
  bool use_sbias = false;
  if constexpr (!QSMOOTH) {
    float smax = 0.f;
    for (int jj = lane; jj <= last; jj += 64) smax = fmaxf(smax, sKh[jj]);
    use_sbias = cq * wave_max_nonneg_f32(smax) < 1e-3f;
  }
  auto run = [&](auto sbias_tag) __attribute__((always_inline)) {
    constexpr bool SBIAS = decltype(sbias_tag)::value;
    v16i sA[2], sB[2];
    fwd_s_mfma<D, SBIAS>(cur, qf, sA, lane);
    // KV128: numerics blocks of 128 keys = pairs of tiles (j even, j + 1).  The row max of the pair must be
    // known before either tile is quantised, so before the even tile the logits of the odd one are formed
    // once just for their row max (8 or 4 MFMAs that nothing overlaps) and dropped; fwd_tile then forms them
    // again under the even tile's softmax as it always does (the matrix pipe has the time, and holding them
    // instead would cost 32 registers this kernel does not have).  The odd tile takes the even tile's own
    // row max, which fwd_tile leaves in `pm`.
    PairMax pm{INT_MIN, -INFINITY};
    float sk = scalar_load(sKh), sv = scalar_load(sVh);     // scales of tile j
    auto partner_max = [&](const int jn, auto mask_tag) __attribute__((always_inline)) {
      constexpr bool MASKED = decltype(mask_tag)::value;
      v16i sT[2];
      fwd_s_mfma<D, SBIAS>(nxt, qf, sT, lane);      // tile jn = j + 1 sits in the next ring slot
      // (with SBIAS the accumulators hold B0 + s: the same order)
      pm = tile_row_max<QSMOOTH, MASKED>(sT, cq * scalar_load(sKh + jn), (const float*)(nxt + BIAS_OFF + wave * 256), jn * kBlock, qlim, h);
    };
    constexpr bool CARRY = !QSMOOTH && !KV128;
    int carried = INT_MIN;
    if (CARRY && last > 0) carried = tile_row_max<false, false>(sA, 0.f, nullptr, 0, 0, h).i;
    auto full_iter = [&](const int j, v16i (&sc)[2], v16i (&sn)[2]) __attribute__((always_inline)) {
      const int jl = min(j + 3, n_tiles - 1);
      asm volatile("" : "+v"(lane16));
      const float skn = scalar_load(sKh + j + 1), svn = scalar_load(sVh + j + 1);     // (j < last: tile j + 1 exists)
      fwd_tile<D, QSMOOTH, false, true, SBIAS, KV128, CARRY>([&](int k) __attribute__((always_inline)) { if (k < CPW) copy_piece(jl, nx3, k); },
                                        nxt, cur + TILE_BYTES, qf, sc, sn, oacc, w_bias, m_ref, l_part,
                                        cq * sk, sv, (const float*)(cur + BIAS_OFF + wave * 256), j * kBlock, q, lane, h, &pm, &carried);
      if ((j & (kBiasPeriod - 1)) == kBiasPeriod - 1) unbias();
      sk = skn;
      sv = svn;
      end_iter(true);
    };
    int j = 0;
    for (; j + 1 < last; j += 2) {
      if constexpr (KV128) partner_max(j + 1, std::false_type{});
      full_iter(j, sA, sB);
      full_iter(j + 1, sB, sA);
    }
    // (j is even here: either the last tile itself, which then has no partner, or the tile before it)
    if constexpr (KV128) pm = PairMax{INT_MIN, -INFINITY};
    if (j < last) {
      if constexpr (KV128) partner_max(j + 1, std::true_type{});
      full_iter(j, sA, sB);
#pragma unroll
      for (int kb = 0; kb < 2; kb++) sA[kb] = sB[kb];
      j++;
    }
    {
      const bool issue = j + 3 < n_tiles;
      if (issue) stage_load(j + 3, nx3);
      // (the last tile always takes the masked path: without the causal mask it hides the keys past nvalid)
      fwd_tile<D, QSMOOTH, true, false, SBIAS, KV128>([](int) {}, nxt, cur + TILE_BYTES, qf, sA, sB, oacc, w_bias, m_ref, l_part,
                                        cq * sk, sv, (const float*)(cur + BIAS_OFF + wave * 256), j * kBlock, qlim, lane, h, &pm);
      end_iter(issue);
      j++;
    }
    for (; j < n_tiles; j++) keep_ring_moving(j);
    unbias();
    // ---- epilogue: O = O / l, L = m + log(l) (l carries a factor 127) ----
    const float l_tot = half_swap_sum_f32(l_part[0]) + half_swap_sum_f32(l_part[1]);
    const float inv_l = 1.0f / l_tot;
    if (q >= args.nq_valid) return;                    // a query row that does not exist
    unsigned short* Oh = args.O + args.oview.row(bh, q);
#pragma unroll
    for (int cb = 0; cb < KS; cb++)
#pragma unroll
      for (int aa = 0; aa < 4; aa++) {
        v4us o;
#pragma unroll
        for (int b = 0; b < 4; b++) o[b] = float_to_bf16_bits(oacc[cb][4 * aa + b] * inv_l);
        *(v4us*)(Oh + 32 * cb + 8 * aa + 4 * h) = o;
      }
    // (LSE is [BH, nq_valid]: the caller's own row count)
    if (h == 0) args.LSE[(size_t)bh * args.nq_valid + q] = (m_ref + __builtin_amdgcn_logf(l_tot) - kLog2_127) * kLn2;
  };
  // (each path runs to the end of the kernel, so that no register state has to be merged)
  if (__builtin_amdgcn_readfirstlane((int)use_sbias)) run(std::true_type{});
  else run(std::false_type{});
}

// ---- two waves per 32 queries ------------------------------------------------------------------------
// sage_fwd_pair_kernel: the forward for calls that do not fill the machine (numerics blocks of 64 keys).  A
// workgroup owns 32 * NQ queries and has 2 * NQ waves: wave (query group qw, half kb) takes the 32-key block kb
// of every tile for the logits and the softmax, and half of the channels for O.  What the two waves of a query
// group owe each other, the row max of their half tile and the P^ codes of it, goes through LDS,
// software-pipelined over one barrier per tile: interval t finishes the softmax of tile t, adds tile t - 1 to O
// and forms S of tile t + 1 with its half row max, so each finds the other wave's part of the interval before.
//
// (Copies that every interval issues, past the last tile ones never read, the inline constant in the products and exponents
// formed a slot ahead of their exp2: 2 heads of N = 4096 63.6 -> 59.1 us a call, 8 of N = 1000 25.6 -> 24.7.)
// Such calls take the time of one wave's chain of tiles: with one wave per SIMD sage_fwd_kernel needs 1.02 us for
// each further tile (2 heads of N = 4096 against 8 of N = 1024, same pre-pass), most of it the wave's own instruction
// issue (one vector instruction in about 4.8 cycles).  Half a tile per wave takes 0.77 us: less than half of the
// instructions are saved (row statistics are formed twice), and the interval is a chain of its own, from the other
// wave's row max in LDS through exp2 and packing to the next one.  The arithmetic of every value and its order are
// those of sage_fwd_kernel, so both give the same bits and the choice may depend on how full the machine is.  (With
// 128 registers, four waves per SIMD, this form was tried for full machines too: 925 us against 756 at
// the headline shape.)
template <int D, bool CAUSAL, bool QSMOOTH, int NQ>
__global__ void __launch_bounds__(128 * NQ, 2) sage_fwd_pair_kernel(FwdArgs args) {
  constexpr int KS = D / 32;
  constexpr int CBW = KS / 2;                                  // channel blocks of O per wave
  constexpr int NW = 2 * NQ;
  constexpr int TILE_BYTES = 64 * D;
  constexpr int PAIR = 2 * TILE_BYTES;
  constexpr int NFRAG = PAIR / 1024;
  constexpr int SLOT = PAIR + (QSMOOTH ? 256 : 0);             // (one Q block = one bias row per workgroup)
  constexpr int R = 3;
  constexpr int CPW = NFRAG / NW + (QSMOOTH ? 1 : 0);          // copies per wave and slot
  static_assert(NFRAG % NW == 0, "every wave must issue the same number of copies");
  static_assert(NQ * 32 == kBlock, "a workgroup is one Q block: rows of the workspace tensors come in whole blocks");
  // (one LDS object: reads of a second one, which no asynchronous copy writes, would be made to wait for the copies in flight)
  struct Lds {
    int8_t ring[R * SLOT];                                     // slot p: K^ of tile p + 2 | V^ of tile p | biases of tile p + 2
    int8_t pxch[2][NQ][2][1024];                               // [tile parity][query group][key block]: P^ as B operand
    float mxch[2][NQ][2][32];                                  // [tile parity][query group][key block][query]: half row max (bits)
  };
  __shared__ __attribute__((aligned(16))) Lds L;
  auto& ring = L.ring;
  auto& pxch = L.pxch;
  auto& mxch = L.mxch;

  const WorkItem wi = work_item(folded(blockIdx.x, args.fold_end), args.n_qtiles, args.head_set);
  const int bh = wi.head;
  const int qt = args.n_qtiles - 1 - wi.item;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qw = wave >> 1, kb = wave & 1;
  const int ql = lane & 31, h = lane >> 5;
  const int N = args.N;
  const int q0 = (qt * NQ + qw) * 32;
  const int q = q0 + ql;
  const int qlim = CAUSAL ? q + args.shift : args.nvalid - 1;
  const int nblk = N / kBlock;
  const int nqblk = args.Nq / kBlock;
  const int qblk = q0 / kBlock;

  const int8_t* KFh = args.KF + (size_t)bh * N * D;
  const int8_t* VTh = args.VT + (size_t)bh * N * D;
  const float* sKh = args.sK + (size_t)bh * nblk;
  const float* sVh = args.sV + (size_t)bh * nblk;
  const int n_tiles = CAUSAL ? (qt * NQ * 32 + NQ * 32 + args.shift) / kBlock : nblk;
  const int last = n_tiles - 1;                                // (the diagonal block of every wave, with the mask)

  // copies of slot p (K^ of tile p + 2, V^ of tile p; clamped where there is no such tile: never read)
  unsigned lane16 = lane * 16;
  static_assert(NFRAG / 2 % NW == 0, "a copy is of K^ for every wave, or of V^");
  auto copy_piece = [&](int p, int8_t* dst, int k) __attribute__((always_inline)) {
    const int o = wave + NW * k;                               // wave-uniform
    const int jk = min(p + 2, nblk - 1), jv = min(max(p, 0), nblk - 1);
    if (k < NFRAG / 2 / NW) copy_16(uniform(KFh + (size_t)jk * TILE_BYTES + o * 1024) + lane16, dst + o * 1024);
    else if (k < NFRAG / NW) copy_16(uniform(VTh + (size_t)jv * TILE_BYTES + (o - NFRAG / 2) * 1024) + lane16, dst + o * 1024);
    // (every wave copies the row, so that all issue the same number)
    else if (QSMOOTH && k == NFRAG / NW) copy_4(uniform(args.bias + ((size_t)bh * nqblk + qblk) * N + jk * kBlock) + (lane16 >> 2), dst + PAIR);
  };
  int8_t* rd = ring;                                           // slot t - 1
  int8_t* mid = ring + SLOT;                                   // slot t
  int8_t* wr = ring + 2 * SLOT;                                // slot t + 1
#pragma unroll
  for (int k = 0; k < CPW; k++) copy_piece(-1, rd, k);
#pragma unroll
  for (int k = 0; k < CPW; k++) copy_piece(0, mid, k);

  v4i qf[KS];
  {
    const int8_t* p = args.QF + (size_t)bh * args.Nq * D + (size_t)(q0 / 32) * KS * 1024 + lane * 16;
#pragma unroll
    for (int s = 0; s < KS; s++) qf[s] = *(const v4i*)(p + s * 1024);
  }
  const float cq = args.sQ[(size_t)bh * nqblk + qblk] * args.scale_log2e;

  float oacc[CBW][16];
#pragma unroll
  for (int cb = 0; cb < CBW; cb++)
#pragma unroll
    for (int r = 0; r < 16; r++) oacc[cb][r] = 0.f;
  float w_bias = 0.f, m_ref = -INFINITY, l_part = 0.f, w_prev = 0.f;

  bool use_sbias = false;
  if constexpr (!QSMOOTH) {
    float smax = 0.f;
    for (int jj = lane; jj <= last; jj += 64) smax = fmaxf(smax, sKh[jj]);
    use_sbias = cq * wave_max_nonneg_f32(smax) < 1e-3f;
  }
  auto run = [&](auto sbias_tag) __attribute__((always_inline)) {
    constexpr bool SBIAS = decltype(sbias_tag)::value;
    float mown = 0.f;          // half row max of the tile in hand (bits)

    // half row max of tile j (logits s; with Q-smoothing they become floats in the log2 domain), into LDS
    auto half_max = [&](v16i& s, const int j, const float c, const float* bias_row, auto mask_tag) __attribute__((always_inline)) {
      constexpr bool MASK = decltype(mask_tag)::value;
      if constexpr (!QSMOOTH) {
        int m[2] = {INT_MIN, INT_MIN};
#pragma unroll
        for (int r = 0; r < 16; r++) {
          int v = s[r];
          if constexpr (MASK) {
            const int key = j * kBlock + 32 * kb + 8 * (r >> 2) + 4 * h + (r & 3);
            v = key > qlim ? INT_MIN : v;
            s[r] = v;
          }
          m[r >> 3] = max(m[r >> 3], v);
        }
        mown = __int_as_float(half_swap_max_i32(max(m[0], m[1])));
      } else {
        float m[2] = {-INFINITY, -INFINITY};
#pragma unroll
        for (int aa = 0; aa < 4; aa++) {
          const v4f b4 = *(const v4f*)(bias_row + 32 * kb + 8 * aa + 4 * h);
#pragma unroll
          for (int b = 0; b < 4; b++) {
            float v = __builtin_fmaf((float)s[4 * aa + b], c, b4[b]);
            if constexpr (MASK) {
              const int key = j * kBlock + 32 * kb + 8 * aa + 4 * h + b;
              v = key > qlim ? -INFINITY : v;
            }
            s[4 * aa + b] = __float_as_int(v);
            m[b & 1] = fmaxf(m[b & 1], v);
          }
        }
        mown = half_swap_max_f32(fmaxf(m[0], m[1]));
      }
      mxch[j & 1][qw][kb][ql] = mown;
    };
    auto unbias = [&]() __attribute__((always_inline)) {
      const float corr = kBiasC0 * w_bias;
#pragma unroll
      for (int cb = 0; cb < CBW; cb++)
#pragma unroll
        for (int r = 0; r < 16; r++) oacc[cb][r] -= corr;
      w_bias = 0.f;
    };
    // One interval.  PV / SM / SN: tile t - 1 is added to O, tile t quantised, the logits of tile t + 1 formed.  The
    // vector work of the softmax runs over the matrix work of the other two (P^ does not depend on the running
    // reference); the reference, which scales O, moves after tile t - 1 has been added, as in sage_fwd_kernel.
    auto interval = [&](const int t, const float c, const float sv, const float cn, v16i& s, v16i& sn, auto pv_tag,
                        auto sm_tag, auto sn_tag, auto mask_tag) __attribute__((always_inline)) {
      constexpr bool PV = decltype(pv_tag)::value, SM = decltype(sm_tag)::value, SN = decltype(sn_tag)::value;
      constexpr bool MASK = decltype(mask_tag)::value;
      asm volatile("" : "+v"(lane16));
      const int8_t* kl = rd + kb * KS * 1024 + lane * 16;
      const int8_t* vl = rd + TILE_BYTES + kb * CBW * 1024 + lane * 16;
      float mother = 0.f;
      v4i ka[KS], va[2][CBW], p[2];
      if constexpr (SM) mother = mxch[t & 1][qw][kb ^ 1][ql];
      if constexpr (PV) {
#pragma unroll
        for (int k = 0; k < 2; k++) {
          p[k] = *(const v4i*)(&pxch[(t - 1) & 1][qw][k][lane * 16]);
#pragma unroll
          for (int cb = 0; cb < CBW; cb++) va[k][cb] = *(const v4i*)(vl + (k * KS + cb) * 1024);
        }
      }
      if constexpr (SN) {
#pragma unroll
        for (int k = 0; k < KS; k++) ka[k] = *(const v4i*)(kl + k * 1024);
      }
      __builtin_amdgcn_sched_barrier(0);
      float mloc = 0.f, c_eff = 0.f, off = 0.f;
      if constexpr (SM) {
        float bmax_f = 0.f;
        if constexpr (!QSMOOTH) {
          const int mrow = max(__float_as_int(mown), __float_as_int(mother));
          mloc = (float)(mrow - (SBIAS ? kBiasBits : 0)) * c;
          if constexpr (SBIAS) bmax_f = __int_as_float(mrow);
        } else {
          mloc = fmaxf(mown, mother);
        }
        c_eff = SBIAS ? c * kTwo26 : c;
        off = SBIAS ? __builtin_fmaf(-bmax_f, c_eff, kLog2_127) : kLog2_127 - mloc;
      }
      // exponents of four logits, formed one slot ahead of their exp2
      float xn[4] = {0.f, 0.f, 0.f, 0.f};
      auto form_x = [&](int aa) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < 4; b++) {
          float xv;
          if constexpr (!QSMOOTH) {
            if constexpr (SBIAS) xv = __builtin_fmaf(__int_as_float(s[4 * aa + b]), c_eff, off);
            else xv = __builtin_fmaf((float)s[4 * aa + b], c, off);
            if constexpr (MASK) xv = s[4 * aa + b] == INT_MIN ? -INFINITY : xv;
          } else {
            xv = __int_as_float(s[4 * aa + b]) + off;
          }
          xn[b] = xv;
        }
      };
      if constexpr (SM) form_x(0);
      v16i tt[CBW];
      float psum[4] = {0.f, 0.f, 0.f, 0.f};
      v4i pf;
#pragma unroll
      for (int sl = 0; sl < 5; sl++) {
        // matrix work, one slot behind the vector work (the LDS reads of the operands are under way until then): one
        // step of S (D / 32 of them), one MFMA of P^V^ (2 * CBW)
        if constexpr (SN) {
          const int aa = sl - 1;
          if (aa >= 0 && aa < KS) {
            if (aa == 0) {
              v16i z;
#pragma unroll
              for (int r = 0; r < 16; r++) z[r] = 0;
              sn = SBIAS ? mfma_from_bias(ka[0], qf[0]) : __builtin_amdgcn_mfma_i32_32x32x32_i8(ka[0], qf[0], z, 0, 0, 0);
            } else {
              sn = __builtin_amdgcn_mfma_i32_32x32x32_i8(ka[aa], qf[aa], sn, 0, 0, 0);
            }
          }
        }
        if constexpr (PV) {
          const int aa = sl - 1;
          if (aa >= 0 && aa < 2 * CBW) {
            const int k = aa / CBW, cb = aa % CBW;
            if (k == 0) {
              tt[cb] = mfma_from_bias(va[0][cb], p[0]);
            } else {
              tt[cb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(va[1][cb], p[1], tt[cb], 0, 0, 0);
            }
          }
        }
        if (sl < CPW) copy_piece(t + 1, wr, sl);
        if (SM && sl < 4) {
          const int aa = sl;
          unsigned u = 0;
          float e[4];
#pragma unroll
          for (int b = 0; b < 4; b++) e[b] = __builtin_amdgcn_exp2f(xn[b]);
          __builtin_amdgcn_sched_barrier(0);
          if (aa < 3) form_x(aa + 1);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int b = 0; b < 4; b++) {
            psum[b] = aa == 0 ? e[b] : psum[b] + e[b];
            pin(psum[b]);
            u = __builtin_amdgcn_cvt_pk_u8_f32(e[b], b, u);
          }
          pf[aa] = (int)u;
        }
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int k = 5; k < CPW; k++) copy_piece(t + 1, wr, k);
      if constexpr (SM) *(v4i*)(&pxch[t & 1][qw][kb][lane * 16]) = pf;
      if constexpr (PV) {
#pragma unroll
        for (int cb = 0; cb < CBW; cb++)
#pragma unroll
          for (int r = 0; r < 16; r++) oacc[cb][r] = __builtin_fmaf(__int_as_float(tt[cb][r]), w_prev, oacc[cb][r]);
        if (((t - 1) & (kBiasPeriod - 1)) == kBiasPeriod - 1) unbias();
      }
      if constexpr (SM) {
        if (__builtin_amdgcn_ballot_w64(mloc > m_ref + kTau) != 0) {
          const float m_new = fmaxf(m_ref, mloc);
          const float alpha = __builtin_amdgcn_exp2f(m_ref - m_new);   // 0 on the first tile
          l_part *= alpha;
          w_bias *= alpha;
#pragma unroll
          for (int cb = 0; cb < CBW; cb++)
#pragma unroll
            for (int r = 0; r < 16; r++) oacc[cb][r] *= alpha;
          m_ref = m_new;
        }
        const float beta = __builtin_amdgcn_exp2f(mloc - m_ref);
        l_part = __builtin_fmaf(beta, (psum[0] + psum[1]) + (psum[2] + psum[3]), l_part);
        w_prev = beta * sv * kTwo26;
        w_bias += w_prev;
      }
      if constexpr (SN) half_max(sn, t + 1, cn, (const float*)(rd + PAIR), mask_tag);
      // the copies of slot t (issued one interval ago) have landed; this interval's stay in flight
      __builtin_amdgcn_s_waitcnt(vmcnt_only(CPW));
      barrier_lds_only();
      int8_t* x = rd;
      rd = mid;
      mid = wr;
      wr = x;
    };
    using T = std::true_type;
    using F = std::false_type;

    // tile 0: logits straight from memory
    v16i sA, sB;
    float sk = scalar_load(sKh), sv = scalar_load(sVh);
#pragma unroll
    for (int r = 0; r < 16; r++) sA[r] = SBIAS ? kBiasBits : 0;
#pragma unroll
    for (int k = 0; k < KS; k++)
      sA = __builtin_amdgcn_mfma_i32_32x32x32_i8(*(const v4i*)(KFh + (kb * KS + k) * 1024 + lane * 16), qf[k], sA, 0, 0, 0);
    half_max(sA, 0, cq * sk, QSMOOTH ? args.bias + ((size_t)bh * nqblk + qblk) * N : nullptr, T{});
    barrier_all_memory();

    // interval t with the scales of tiles t (sk, sv) and t + 1 (fetched one interval ahead of their use)
    auto step = [&](const int t, v16i& s, v16i& sn, auto pv_tag, auto sm_tag, auto sn_tag, auto mask_tag) __attribute__((always_inline)) {
      const int jn = min(t + 1, nblk - 1);
      const float skn = scalar_load(sKh + jn), svn = scalar_load(sVh + jn);
      interval(t, cq * sk, sv, cq * skn, s, sn, pv_tag, sm_tag, sn_tag, mask_tag);
      sk = skn;
      sv = svn;
    };
    // (the masked forms leave visible keys as they are)
    int t = 0;
    if (last >= 1) {
      step(t++, sA, sB, F{}, T{}, T{}, T{});
      for (; t + 2 < last; t += 2) {
        step(t, sB, sA, T{}, T{}, T{}, F{});
        step(t + 1, sA, sB, T{}, T{}, T{}, F{});
      }
      for (; t < last; t++) {
        step(t, sB, sA, T{}, T{}, T{}, T{});
        sB = sA;
      }
      step(t++, sB, sA, T{}, T{}, F{}, T{});
      step(t++, sB, sA, T{}, F{}, F{}, F{});
    } else {
      step(t++, sA, sB, F{}, T{}, F{}, T{});
      step(t++, sA, sB, T{}, F{}, F{}, F{});
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_only(0));                 // (the copies past the last tile land before the LDS is given up)
    unbias();
  };
  if (__builtin_amdgcn_readfirstlane((int)use_sbias)) run(std::true_type{});
  else run(std::false_type{});

  // ---- epilogue: O = O / l, L = m + log(l) (l carries a factor 127); the two halves of l meet in LDS ----
  mxch[0][qw][kb][ql] = half_swap_sum_f32(l_part);
  barrier_lds_only();
  if (q >= args.nq_valid) return;                              // a query row that does not exist
  const float l_tot = mxch[0][qw][0][ql] + mxch[0][qw][1][ql];
  const float inv_l = 1.0f / l_tot;
  unsigned short* Oh = args.O + args.oview.row(bh, q);
#pragma unroll
  for (int cb = 0; cb < CBW; cb++)
#pragma unroll
    for (int aa = 0; aa < 4; aa++) {
      v4us o;
#pragma unroll
      for (int b = 0; b < 4; b++) o[b] = float_to_bf16_bits(oacc[cb][4 * aa + b] * inv_l);
      *(v4us*)(Oh + 32 * (kb * CBW + cb) + 8 * aa + 4 * h) = o;
    }
  if (kb == 0 && h == 0) args.LSE[(size_t)bh * args.nq_valid + q] = (m_ref + __builtin_amdgcn_logf(l_tot) - kLog2_127) * kLn2;
}

// What the copies of sage_fwd_quad_kernel read for slot p, in bytes from the head's codes: K^ of tile 0 or 1 of pair p + 2, V^ of pair p;
// the head's last tile (at `last`) where there is no such tile.  (Host code too: a test goes through every copy.)
__host__ __device__ inline int quad_k_offset(int p, int tile, int tile_bytes, int last) {
  const int o = (2 * p + 4 + tile) * tile_bytes;
  return o < last ? o : last;
}
__host__ __device__ inline int quad_v_offset(int p, int tile, int tile_bytes, int last) {
  const int t = 2 * p + tile, o = (t > 0 ? t : 0) * tile_bytes;
  return o < last ? o : last;
}
// Block whose scale interval t loads for tile 0 or 1 of pair t + 1: two blocks at a time, so the second may be one past the head's last.
__host__ __device__ inline int quad_scale_block(int t) { return 2 * t + 2; }

// ---- four waves per 32 queries -----------------------------------------------------------------------
// sage_fwd_quad_kernel: the same for calls that leave half of the SIMDs idle even then.  A workgroup is one Q block, eight waves;
// the four waves of 32 queries take TWO tiles at a time, wave (tile, key block) one 32-key block of the pair, and a quarter of O's
// channels each (d = 64: half of them, twice over).  An interval is as long a chain as above and there are half as many.  The tiles
// of a pair are added to O one after the other by every wave, and the sums of P of either key block in the order of the tiles, so
// the bits are those of the other two kernels: row maxima, P^ and the sums of P go through LDS for that.
//
// What an interval (0.85 us) takes is each wave's own instruction stream and its waits.  The steps, 1 and 4 heads of N = 4096, whole
// calls, two waves per 32 queries 51.8, 56.6 us: four waves 44.9, 48.7; copies whose addresses are one scalar minimum away and
// scales loaded behind the first waits for LDS (85 -> 35 scalar instructions an interval, and such a wait no longer waits for all)
// 42.7, 47.0; the operands of the coming interval's products read under the end of this one 41.3, 45.5.  Others: 8 heads of N = 1000
// 23.4 -> 21.5, 16 of 1024 25.8 -> 23.7, 8 of 2048 without the mask 35.2 -> 30.9.
template <int D, bool CAUSAL, bool QSMOOTH>
__global__ void __launch_bounds__(512, 1) sage_fwd_quad_kernel(FwdArgs args) {
  constexpr int KS = D / 32;
  constexpr int NQ = 2, NW = 4 * NQ;
  constexpr int TILE_BYTES = 64 * D;
  constexpr int PAIR = 2 * TILE_BYTES;
  constexpr int TF = TILE_BYTES / 1024;                        // fragments of a tile
  constexpr int NFRAG = 2 * PAIR / 1024;
  constexpr int SLOT = 2 * PAIR + (QSMOOTH ? 512 : 0);         // (one Q block = one bias row per workgroup)
  constexpr int R = 3;
  constexpr int CPW = NFRAG / NW + (QSMOOTH ? 1 : 0);          // copies per wave and slot
  static_assert(NFRAG % NW == 0, "every wave must issue the same number of copies");
  static_assert(NQ * 32 == kBlock, "a workgroup is one Q block: rows of the workspace tensors come in whole blocks");
  // (one LDS object: reads of a second one, which no asynchronous copy writes, would be made to wait for the copies in flight)
  struct Lds {
    int8_t ring[R * SLOT];                                     // slot p: K^ of pair p + 2 | V^ of pair p | biases of pair p + 1
    int8_t pxch[2][NQ][4][1024];                               // [parity of the pair][query group][key block]: P^ as B operand
    float sxch[2][NQ][4][64];                                  // [..][lane]: the lane's sum of P
    float mxch[2][NQ][4][32];                                  // [..][query]: row max over the key block (bits)
  };
  __shared__ __attribute__((aligned(16))) Lds L;
  auto& ring = L.ring;
  auto& pxch = L.pxch;
  auto& mxch = L.mxch;
  auto& sxch = L.sxch;

  const WorkItem wi = work_item(blockIdx.x, args.n_qtiles, args.head_set);
  const int bh = wi.head;
  const int qt = args.n_qtiles - 1 - wi.item;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qw = wave >> 2, w4 = wave & 3;
  const int tp = w4 >> 1, kb = w4 & 1;                         // tile of a pair, key block of it
  const int cb = w4 % KS;                                      // channel block of O (d = 64: two waves form each)
  const int ql = lane & 31, h = lane >> 5;
  const int N = args.N;
  const int q0 = (qt * NQ + qw) * 32;
  const int q = q0 + ql;
  const int qlim = CAUSAL ? q + args.shift : args.nvalid - 1;
  const int nblk = N / kBlock;
  const int nqblk = args.Nq / kBlock;
  const int qblk = q0 / kBlock;

  const int8_t* KFh = args.KF + (size_t)bh * N * D;
  const int8_t* VTh = args.VT + (size_t)bh * N * D;
  const float* sKh = args.sK + (size_t)bh * nblk;
  const float* sVh = args.sV + (size_t)bh * nblk;
  const int n_tiles = CAUSAL ? (qt * NQ * 32 + NQ * 32 + args.shift) / kBlock : nblk;
  const int last = n_tiles - 1;                                // (the diagonal block of every wave, with the mask)
  const int n_pairs = (n_tiles + 1) / 2;

  // Copies of slot p: K^ of pair p + 2, V^ of pair p (from the last tile where there is no such tile: K^ is masked, V^ never used).
  // One lane offset serves all of a wave's copies, and a copy is a minimum and an addition of scalars away: the wave's own
  // instruction stream is what such a call takes.
  constexpr int KC = NFRAG / 2 / NW;                           // copies of K^ per wave and slot, as many of V^
  static_assert(NFRAG / 2 % NW == 0 && (KC == 2 || TF == NW / 2), "a copy is of K^ for every wave, or of V^; of one tile");
  // (raw buffers of the head's codes: the descriptor's last word has the 32-bit float format, no swizzle and no index; past N * D bytes
  // they read zeros)
  const __amdgpu_buffer_rsrc_t krs = __builtin_amdgcn_make_buffer_rsrc((void*)KFh, 0, N * D, 0x27000);
  const __amdgpu_buffer_rsrc_t vrs = __builtin_amdgcn_make_buffer_rsrc((void*)VTh, 0, N * D, 0x27000);
  unsigned lane_off = lane * 16 + (wave % TF) * 1024;
  const int last_off = (nblk - 1) * TILE_BYTES;
  auto copy_piece = [&](int p, int8_t* dst, int k) __attribute__((always_inline)) {
    const int o = wave + NW * k;                               // wave-uniform
    const int tile = KC == 2 ? k % KC : wave / TF;
    if (k < KC) {
      __builtin_amdgcn_raw_ptr_buffer_load_lds(krs, (lptr_t)(dst + o * 1024), 16, lane_off, quad_k_offset(p, tile, TILE_BYTES, last_off), 0, 0);
    } else if (k < 2 * KC) {
      __builtin_amdgcn_raw_ptr_buffer_load_lds(vrs, (lptr_t)(dst + o * 1024), 16, lane_off, quad_v_offset(p, tile, TILE_BYTES, last_off), 0, 0);
    } else if (QSMOOTH && k == 2 * KC) {
      // (every wave copies a row, so that all issue the same number)
      copy_4(uniform(args.bias + ((size_t)bh * nqblk + qblk) * N + min(max(2 * p + 2 + (wave & 1), 0), nblk - 1) * kBlock) + 4 * lane, dst + 2 * PAIR + (wave & 1) * 256);
    }
  };
  int8_t* rd = ring + SLOT;                                    // slot t
  int8_t* mid = ring + 2 * SLOT;                               // slot t + 1
  int8_t* wr = ring;                                           // slot t + 2 (before: t - 1)
#pragma unroll
  for (int k = 0; k < CPW; k++) copy_piece(-1, wr, k);
#pragma unroll
  for (int k = 0; k < CPW; k++) copy_piece(0, rd, k);
#pragma unroll
  for (int k = 0; k < CPW; k++) copy_piece(1, mid, k);

  v4i qf[KS];
  {
    const int8_t* p = args.QF + (size_t)bh * args.Nq * D + (size_t)(q0 / 32) * KS * 1024 + lane * 16;
#pragma unroll
    for (int s = 0; s < KS; s++) qf[s] = *(const v4i*)(p + s * 1024);
  }
  const float cq = args.sQ[(size_t)bh * nqblk + qblk] * args.scale_log2e;

  float oacc[16];
#pragma unroll
  for (int r = 0; r < 16; r++) oacc[r] = 0.f;
  float w_bias = 0.f, m_ref = -INFINITY, l_part = 0.f;
  float m_prev[2] = {0.f, 0.f};                                // row maxima of the tiles of the pair that is to be added to O

  bool use_sbias = false;
  if constexpr (!QSMOOTH) {
    float smax = 0.f;
    for (int jj = lane; jj <= last; jj += 64) smax = fmaxf(smax, sKh[jj]);
    use_sbias = cq * wave_max_nonneg_f32(smax) < 1e-3f;
  }
  auto run = [&](auto sbias_tag) __attribute__((always_inline)) {
    constexpr bool SBIAS = decltype(sbias_tag)::value;
    // row max over the wave's key block of tile j (logits s; with Q-smoothing they become floats in the log2 domain), into LDS
    auto half_max = [&](v16i& s, const int pair, const float c, const float* bias_row, auto mask_tag) __attribute__((always_inline)) {
      constexpr bool MASK = decltype(mask_tag)::value;
      const int j = 2 * pair + tp;
      float mown;
      if constexpr (!QSMOOTH) {
        int m[2] = {INT_MIN, INT_MIN};
#pragma unroll
        for (int r = 0; r < 16; r++) {
          int v = s[r];
          if constexpr (MASK) {
            const int key = j * kBlock + 32 * kb + 8 * (r >> 2) + 4 * h + (r & 3);
            v = key > qlim ? INT_MIN : v;
            s[r] = v;
          }
          m[r >> 3] = max(m[r >> 3], v);
        }
        mown = __int_as_float(half_swap_max_i32(max(m[0], m[1])));
      } else {
        float m[2] = {-INFINITY, -INFINITY};
#pragma unroll
        for (int aa = 0; aa < 4; aa++) {
          const v4f b4 = *(const v4f*)(bias_row + 32 * kb + 8 * aa + 4 * h);
#pragma unroll
          for (int b = 0; b < 4; b++) {
            float v = __builtin_fmaf((float)s[4 * aa + b], c, b4[b]);
            if constexpr (MASK) {
              const int key = j * kBlock + 32 * kb + 8 * aa + 4 * h + b;
              v = key > qlim ? -INFINITY : v;
            }
            s[4 * aa + b] = __float_as_int(v);
            m[b & 1] = fmaxf(m[b & 1], v);
          }
        }
        mown = half_swap_max_f32(fmaxf(m[0], m[1]));
      }
      mxch[pair & 1][qw][w4][ql] = mown;
    };
    auto unbias = [&]() __attribute__((always_inline)) {
      const float corr = kBiasC0 * w_bias;
#pragma unroll
      for (int r = 0; r < 16; r++) oacc[r] -= corr;
      w_bias = 0.f;
    };
    // The running reference for a tile of row max mloc, and the sum of its P; returns the weight of its P^V^.
    auto take_tile = [&](const float mloc, const float psum, const float sv) __attribute__((always_inline)) {
      if (__builtin_amdgcn_ballot_w64(mloc > m_ref + kTau) != 0) {
        const float m_new = fmaxf(m_ref, mloc);
        const float alpha = __builtin_amdgcn_exp2f(m_ref - m_new);     // 0 on the first tile
        l_part *= alpha;
        w_bias *= alpha;
#pragma unroll
        for (int r = 0; r < 16; r++) oacc[r] *= alpha;
        m_ref = m_new;
      }
      const float beta = __builtin_amdgcn_exp2f(mloc - m_ref);
      l_part = __builtin_fmaf(beta, psum, l_part);
      const float w = beta * sv * kTwo26;
      w_bias += w;
      return w;
    };
    // scales of the tiles of pairs t (sk, sv) and t - 1 (svp).  (Two at a time; past the head's last tile it is whatever lies behind
    // them in the workspace, which has the codes behind the scales, and multiplies masked logits or nothing.)
    v2f sk = scalar_load2(sKh), sv = scalar_load2(sVh), svp = {0.f, 0.f};
    // K^ of pair t + 1 and V^ of pair t - 1 for interval t, read under the end of the interval before
    v4i ka[KS], va[2][2];
    auto read_operands = [&](const int8_t* slot) __attribute__((always_inline)) {
      const int8_t* kl = slot + tp * TILE_BYTES + kb * KS * 1024 + lane * 16;
      const int8_t* vl = slot + PAIR + cb * 1024 + lane * 16;
#pragma unroll
      for (int k = 0; k < KS; k++) ka[k] = *(const v4i*)(kl + k * 1024);
#pragma unroll
      for (int k = 0; k < 2; k++)
#pragma unroll
        for (int u = 0; u < 2; u++) va[u][k] = *(const v4i*)(vl + u * TILE_BYTES + k * KS * 1024);
    };
    // One interval.  PV / SM / SN: pair t - 1 is added to O, tile after tile, pair t quantised, the logits of pair t + 1 formed.
    auto interval = [&](const int t, v16i& s, v16i& sn, auto pv_tag, auto sm_tag, auto sn_tag, auto mask_tag) __attribute__((always_inline)) {
      constexpr bool PV = decltype(pv_tag)::value, SM = decltype(sm_tag)::value, SN = decltype(sn_tag)::value;
      constexpr bool MASK = decltype(mask_tag)::value;
      asm volatile("" : "+v"(lane_off));
      const float c[2] = {cq * sk[0], cq * sk[1]};
      v2f skn = sk, svn = sv;
      float mx[4], ps[2];
      v4i p[2][2];
      if constexpr (SM) {
#pragma unroll
        for (int k = 0; k < 4; k++) mx[k] = mxch[t & 1][qw][k][ql];
      }
      if constexpr (PV) {
#pragma unroll
        for (int u = 0; u < 2; u++) {
          ps[u] = sxch[(t - 1) & 1][qw][2 * u + kb][lane];
#pragma unroll
          for (int k = 0; k < 2; k++) p[u][k] = *(const v4i*)(&pxch[(t - 1) & 1][qw][2 * u + k][lane * 16]);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      float m_pair[2] = {0.f, 0.f}, c_own = 0.f, c_eff = 0.f, off = 0.f;
      if constexpr (SM) {
        float bmax_f = 0.f;
        c_own = tp ? c[1] : c[0];
#pragma unroll
        for (int u = 0; u < 2; u++) {
          if constexpr (!QSMOOTH) {
            const int mrow = max(__float_as_int(mx[2 * u]), __float_as_int(mx[2 * u + 1]));
            m_pair[u] = (float)(mrow - (SBIAS ? kBiasBits : 0)) * c[u];
            if constexpr (SBIAS) bmax_f = tp == u ? __int_as_float(mrow) : bmax_f;
          } else {
            m_pair[u] = fmaxf(mx[2 * u], mx[2 * u + 1]);
          }
        }
        c_eff = SBIAS ? c_own * kTwo26 : c_own;
        off = SBIAS ? __builtin_fmaf(-bmax_f, c_eff, kLog2_127) : kLog2_127 - (tp ? m_pair[1] : m_pair[0]);
      }
      // exponents of four logits, formed one slot ahead of their exp2
      float xn[4] = {0.f, 0.f, 0.f, 0.f};
      auto form_x = [&](int aa) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < 4; b++) {
          float xv;
          if constexpr (!QSMOOTH) {
            if constexpr (SBIAS) xv = __builtin_fmaf(__int_as_float(s[4 * aa + b]), c_eff, off);
            else xv = __builtin_fmaf((float)s[4 * aa + b], c_own, off);
            if constexpr (MASK) xv = s[4 * aa + b] == INT_MIN ? -INFINITY : xv;
          } else {
            xv = __int_as_float(s[4 * aa + b]) + off;
          }
          xn[b] = xv;
        }
      };
      if constexpr (SM) form_x(0);
      v16i tt[2];
      float psum[4] = {0.f, 0.f, 0.f, 0.f};
      v4i pf;
#pragma unroll
      for (int sl = 0; sl < 5; sl++) {
        // matrix work: one step of S (D / 32 of them) and, a slot behind (P^ is under way until then), one product of P^V^
        if constexpr (SN) {
          const int aa = sl;
          if (aa >= 0 && aa < KS) {
            if (aa == 0) {
              v16i z;
#pragma unroll
              for (int r = 0; r < 16; r++) z[r] = 0;
              sn = SBIAS ? mfma_from_bias(ka[0], qf[0]) : __builtin_amdgcn_mfma_i32_32x32x32_i8(ka[0], qf[0], z, 0, 0, 0);
            } else {
              sn = __builtin_amdgcn_mfma_i32_32x32x32_i8(ka[aa], qf[aa], sn, 0, 0, 0);
            }
          }
        }
        if constexpr (PV) {
          const int aa = sl - 1;
          if (aa >= 0) {
            const int k = aa / 2, u = aa % 2;
            tt[u] = k == 0 ? mfma_from_bias(va[u][0], p[u][0]) : __builtin_amdgcn_mfma_i32_32x32x32_i8(va[u][1], p[u][1], tt[u], 0, 0, 0);
          }
        }
        // (behind the first waits for LDS: scalar loads come back out of order, and with one under way every such wait is for all)
        if (SN && sl == 1) {
          skn = scalar_load2(sKh + quad_scale_block(t));
          svn = scalar_load2(sVh + quad_scale_block(t));
        }
        if (sl < CPW) copy_piece(t + 2, wr, sl);
        if (SM && sl < 4) {
          const int aa = sl;
          unsigned u = 0;
          float e[4];
#pragma unroll
          for (int b = 0; b < 4; b++) e[b] = __builtin_amdgcn_exp2f(xn[b]);
          __builtin_amdgcn_sched_barrier(0);
          if (aa < 3) form_x(aa + 1);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int b = 0; b < 4; b++) {
            psum[b] = aa == 0 ? e[b] : psum[b] + e[b];
            pin(psum[b]);
            u = __builtin_amdgcn_cvt_pk_u8_f32(e[b], b, u);
          }
          pf[aa] = (int)u;
        }
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int k = 5; k < CPW; k++) copy_piece(t + 2, wr, k);
      read_operands(rd);
      if constexpr (SN) half_max(sn, t + 1, cq * (tp ? skn[1] : skn[0]), (const float*)(rd + 2 * PAIR + tp * 256), mask_tag);
      if constexpr (SM) {
        *(v4i*)(&pxch[t & 1][qw][w4][lane * 16]) = pf;
        sxch[t & 1][qw][w4][lane] = (psum[0] + psum[1]) + (psum[2] + psum[3]);
      }
      if constexpr (PV) {
        auto add = [&](const v16i& x, const float w) __attribute__((always_inline)) {
#pragma unroll
          for (int r = 0; r < 16; r++) oacc[r] = __builtin_fmaf(__int_as_float(x[r]), w, oacc[r]);
        };
        add(tt[0], take_tile(m_prev[0], ps[0], svp[0]));
        if (!MASK || 2 * t - 1 <= last) {
          add(tt[1], take_tile(m_prev[1], ps[1], svp[1]));
          if (((2 * t - 1) & (kBiasPeriod - 1)) == kBiasPeriod - 1) unbias();
        }
      }
      if constexpr (SM) {
        m_prev[0] = m_pair[0];
        m_prev[1] = m_pair[1];
      }
      // the copies of slot t + 1 (issued one interval ago) have landed; this interval's stay in flight
      __builtin_amdgcn_s_waitcnt(vmcnt_only(CPW));
      barrier_lds_only();
      svp = sv;
      sk = skn;
      sv = svn;
      int8_t* x = rd;
      rd = mid;
      mid = wr;
      wr = x;
    };
    using T = std::true_type;
    using F = std::false_type;

    // pair 0: logits straight from memory
    v16i sA, sB;
    const int j0 = min(tp, nblk - 1);
#pragma unroll
    for (int r = 0; r < 16; r++) sA[r] = SBIAS ? kBiasBits : 0;
#pragma unroll
    for (int k = 0; k < KS; k++)
      sA = __builtin_amdgcn_mfma_i32_32x32x32_i8(*(const v4i*)(KFh + (size_t)j0 * TILE_BYTES + (kb * KS + k) * 1024 + lane * 16), qf[k], sA, 0, 0, 0);
    half_max(sA, 0, cq * (tp ? sk[1] : sk[0]), QSMOOTH ? args.bias + ((size_t)bh * nqblk + qblk) * N + j0 * kBlock : nullptr, T{});
    barrier_all_memory();
    read_operands(wr);
    barrier_lds_only();        // (interval 0 copies there)

    // (the masked forms leave visible keys as they are)
    const int lp = n_pairs - 1;
    int t = 0;
    if (lp >= 1) {
      interval(t++, sA, sB, F{}, T{}, T{}, T{});
      for (; t + 2 < lp; t += 2) {
        interval(t, sB, sA, T{}, T{}, T{}, F{});
        interval(t + 1, sA, sB, T{}, T{}, T{}, F{});
      }
      for (; t < lp; t++) {
        interval(t, sB, sA, T{}, T{}, T{}, T{});
        sB = sA;
      }
      interval(t++, sB, sA, T{}, T{}, F{}, T{});
      interval(t++, sB, sA, T{}, F{}, F{}, T{});
    } else {
      interval(t++, sA, sB, F{}, T{}, F{}, T{});
      interval(t++, sA, sB, T{}, F{}, F{}, T{});
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_only(0));                 // (the copies past the last tile land before the LDS is given up)
    unbias();
  };
  if (__builtin_amdgcn_readfirstlane((int)use_sbias)) run(std::true_type{});
  else run(std::false_type{});

  // ---- epilogue: O = O / l, L = m + log(l) (l carries a factor 127); the two halves of l meet in LDS ----
  mxch[0][qw][w4][ql] = half_swap_sum_f32(l_part);
  barrier_lds_only();
  if (q >= args.nq_valid) return;                              // a query row that does not exist
  const float l_tot = mxch[0][qw][0][ql] + mxch[0][qw][1][ql];
  const float inv_l = 1.0f / l_tot;
  unsigned short* Oh = args.O + args.oview.row(bh, q);
  if (w4 < KS) {
#pragma unroll
    for (int aa = 0; aa < 4; aa++) {
      v4us o;
#pragma unroll
      for (int b = 0; b < 4; b++) o[b] = float_to_bf16_bits(oacc[4 * aa + b] * inv_l);
      *(v4us*)(Oh + 32 * cb + 8 * aa + 4 * h) = o;
    }
  }
  if (w4 == 0 && h == 0) args.LSE[(size_t)bh * args.nq_valid + q] = (m_ref + __builtin_amdgcn_logf(l_tot) - kLog2_127) * kLn2;
}

// ---- few query rows against many keys ----------------------------------------------------------------
// A workgroup of 8 waves = NQ groups of 32 queries x NS splits of the keys.  Every wave walks its own
// contiguous range of the workgroup's KV tiles with the arithmetic of sage_fwd_kernel; the partial (O, m, l)
// of the splits meet in LDS at the end, each split finishing a share of the channels.
//
// Where the queries alone do not fill the machine (chunked prefill, cross attention), the time is one wave's chain
// of tiles, about 1 us each; splitting the keys shortens it NS times and puts two waves on every SIMD.  512
// queries x 32 heads against 4096 keys, d = 128: 70 -> 34 us.  (On a full machine the merge and
// the barrier over 8 waves make it the slower form by 5 to 15 %.)  The order of the sums differs from
// sage_fwd_kernel's, which is why square attention does not come here: a head of it gets the same bits alone and in
// any batch.
//
// At d = 128 the ring has two slots per split, so every iteration waits for all of its copies; four would not fit beside
// four splits.
//
// Slot p of a split's ring holds K^ of its tile p + 1 and V^ of its tile p (what iteration p reads: the logits
// of the next tile are formed under the softmax of this one); K^ of the first tile comes straight from memory.
template <int D, bool CAUSAL, bool QSMOOTH, int NQ, int NS>
__global__ void __launch_bounds__(512, 1) sage_fwd_split_kernel(FwdArgs args) {
  constexpr int KS = D / 32;
  constexpr int TILE_BYTES = 64 * D;
  constexpr int PAIR = 2 * TILE_BYTES;
  constexpr int NFRAG = PAIR / 1024;
  constexpr int SLOT = PAIR + (QSMOOTH ? NQ * 256 : 0);
  constexpr int R = NS * 4 * PAIR <= 128 * 1024 ? 4 : 2;       // ring slots per split
  constexpr int CPW = NFRAG / NQ + (QSMOOTH ? 1 : 0);
  static_assert(NQ * NS == 8 && NFRAG % NQ == 0, "8 waves, the same number of copies for each");
  static_assert(NQ * 32 == kBlock, "a workgroup is one Q block: rows of the workspace tensors come in whole blocks");
  constexpr int RING = NS * R * SLOT;
  constexpr int XCH = NQ * NS * KS * 4096;                     // partial O of every wave: [q][split][channel block] x 4 KiB
  __shared__ __attribute__((aligned(16))) int8_t lds[RING > XCH ? RING : XCH];
  __shared__ v2f ml[NQ * NS * 32];                             // (m, l) of every wave and query

  const WorkItem wi = work_item(blockIdx.x, args.n_qtiles, args.head_set);
  const int bh = wi.head;
  const int qt = args.n_qtiles - 1 - wi.item;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qw = wave % NQ, g = wave / NQ;
  const int ql = lane & 31, h = lane >> 5;
  const int N = args.N;
  const int q0 = (qt * NQ + qw) * 32;
  const int q = q0 + ql;
  const int qlim = CAUSAL ? q + args.shift : args.nvalid - 1;
  const int nblk = N / kBlock;
  const int nqblk = args.Nq / kBlock;
  const int qblk = q0 / kBlock;

  const int8_t* KFh = args.KF + (size_t)bh * N * D;
  const int8_t* VTh = args.VT + (size_t)bh * N * D;
  const float* sKh = args.sK + (size_t)bh * nblk;
  const float* sVh = args.sV + (size_t)bh * nblk;

  // this workgroup's tiles, this split's share [a, b) of them (none for the last splits of some counts), its last tile
  const int n_tiles = CAUSAL ? (qt * NQ * 32 + NQ * 32 + args.shift) / kBlock : nblk;
  const int share = (n_tiles + NS - 1) / NS;
  const int a = g * share, b = min(n_tiles, a + share);
  const int last = b - 1;
  const int ac = min(a, nblk - 1);                             // (a split without tiles still reads in bounds)

  v4i qf[KS];
  {
    const int8_t* p = args.QF + (size_t)bh * args.Nq * D + (size_t)(q0 / 32) * KS * 1024 + lane * 16;
#pragma unroll
    for (int s = 0; s < KS; s++) qf[s] = *(const v4i*)(p + s * 1024);
  }
  const float cq = args.sQ[(size_t)bh * nqblk + qblk] * args.scale_log2e;
  const float* bias_row = QSMOOTH ? args.bias + ((size_t)bh * nqblk + qblk) * N : nullptr;

  float oacc[KS][16];
#pragma unroll
  for (int cb = 0; cb < KS; cb++)
#pragma unroll
    for (int r = 0; r < 16; r++) oacc[cb][r] = 0.f;
  float w_bias = 0.f, m_ref = -INFINITY, l_part[2] = {0.f, 0.f};

  int8_t* ring = lds + g * R * SLOT;
  unsigned lane16 = lane * 16;
  static_assert(NFRAG / 2 % NQ == 0, "a copy is of K^ for every wave, or of V^");
  // (slots past the split's tiles are filled with tiles that exist and never read: every iteration issues the same copies)
  auto copy_piece = [&](int p, int k) __attribute__((always_inline)) {
    int8_t* dst = ring + (p % R) * SLOT;
    const int o = qw + NQ * k;
    if (k < NFRAG / 2 / NQ) copy_16(uniform(KFh + (size_t)min(a + p + 1, nblk - 1) * TILE_BYTES + o * 1024) + lane16, dst + o * 1024);
    else if (k < NFRAG / NQ) copy_16(uniform(VTh + (size_t)min(a + p, nblk - 1) * TILE_BYTES + (o - NFRAG / 2) * 1024) + lane16, dst + o * 1024);
    else if (QSMOOTH && k == NFRAG / NQ) copy_4(uniform(bias_row + min(a + p, nblk - 1) * kBlock) + (lane16 >> 2), dst + PAIR + qw * 256);
  };
#pragma unroll
  for (int p = 0; p < R - 1; p++)
#pragma unroll
    for (int k = 0; k < CPW; k++) copy_piece(p, k);
  // end of iteration t: the copies of slot t + 1 have landed (those of younger slots stay in flight)
  auto end_iter = [&]() {
    if constexpr (R > 2) {
      __builtin_amdgcn_s_waitcnt(vmcnt_only((R - 2) * CPW));
      barrier_lds_only();
    } else {
      barrier_all_memory();
    }
  };
  auto unbias = [&]() {
    const float corr = kBiasC0 * w_bias;
#pragma unroll
    for (int cb = 0; cb < KS; cb++)
#pragma unroll
      for (int r = 0; r < 16; r++) oacc[cb][r] -= corr;
    w_bias = 0.f;
  };
  bool use_sbias = false;
  if constexpr (!QSMOOTH) {
    float smax = 0.f;
    for (int jj = a + lane; jj < b; jj += 64) smax = fmaxf(smax, sKh[jj]);
    use_sbias = cq * wave_max_nonneg_f32(smax) < 1e-3f;
  }
  auto run = [&](auto sbias_tag) __attribute__((always_inline)) {
    constexpr bool SBIAS = decltype(sbias_tag)::value;
    v16i sA[2], sB[2];
    fwd_s_mfma<D, SBIAS>(KFh + (size_t)ac * TILE_BYTES, qf, sA, lane);
    barrier_all_memory();                                      // the first slots have landed
    float sk = scalar_load(sKh + ac), sv = scalar_load(sVh + ac);
    constexpr bool CARRY = !QSMOOTH;
    int carried = INT_MIN;
    if constexpr (CARRY) carried = tile_row_max<false, false>(sA, 0.f, nullptr, 0, 0, h).i;
    auto full_iter = [&](const int t, v16i (&sc)[2], v16i (&sn)[2]) __attribute__((always_inline)) {
      asm volatile("" : "+v"(lane16));
      const float skn = scalar_load(sKh + a + t + 1), svn = scalar_load(sVh + a + t + 1);
      const int8_t* slot = ring + (t % R) * SLOT;
      fwd_tile<D, QSMOOTH, false, true, SBIAS, false, CARRY>([&](int k) __attribute__((always_inline)) { if (k < CPW) copy_piece(t + R - 1, k); },
                                               slot, slot + TILE_BYTES, qf, sc, sn, oacc, w_bias, m_ref, l_part, cq * sk, sv,
                                               (const float*)(slot + PAIR + qw * 256), (a + t) * kBlock, q, lane, h, nullptr, &carried);
      if ((t & (kBiasPeriod - 1)) == kBiasPeriod - 1) unbias();
      sk = skn;
      sv = svn;
      end_iter();
    };
    int t = 0;
    for (; a + t + 1 < last; t += 2) {
      full_iter(t, sA, sB);
      full_iter(t + 1, sB, sA);
    }
    if (a + t < last) {
      full_iter(t, sA, sB);
#pragma unroll
      for (int kb = 0; kb < 2; kb++) sA[kb] = sB[kb];
      t++;
    }
    if (a + t <= last) {
      // the split's last tile takes the masked path (which leaves visible keys as they are)
#pragma unroll
      for (int k = 0; k < CPW; k++) copy_piece(t + R - 1, k);
      const int8_t* slot = ring + (t % R) * SLOT;
      fwd_tile<D, QSMOOTH, true, false, SBIAS>([](int) {}, slot, slot + TILE_BYTES, qf, sA, sB, oacc, w_bias, m_ref, l_part, cq * sk, sv,
                                               (const float*)(slot + PAIR + qw * 256), (a + t) * kBlock, qlim, lane, h);
      end_iter();
      t++;
    }
    for (; t < share; t++) {                                   // (a shorter split: every wave meets `share` barriers)
#pragma unroll
      for (int k = 0; k < CPW; k++) copy_piece(t + R - 1, k);
      end_iter();
    }
    if constexpr (R > 2) barrier_all_memory();                 // (the ring is drained before it is used again)
    unbias();
  };
  if (__builtin_amdgcn_readfirstlane((int)use_sbias)) run(std::true_type{});
  else run(std::false_type{});

  // ---- the splits meet: split s finishes the channel blocks cb with cb % NS == s (the ring is drained) ----
  const float l_tot = half_swap_sum_f32(l_part[0]) + half_swap_sum_f32(l_part[1]);
  float* xch = (float*)lds;
#pragma unroll
  for (int cb = 0; cb < KS; cb++)
    if (cb % NS != g) {
#pragma unroll
      for (int aa = 0; aa < 4; aa++)
        *(v4f*)(xch + ((((qw * NS + g) * KS + cb) * 4 + aa) * 64 + lane) * 4) =
            v4f{oacc[cb][4 * aa], oacc[cb][4 * aa + 1], oacc[cb][4 * aa + 2], oacc[cb][4 * aa + 3]};
    }
  if (h == 0) ml[(qw * NS + g) * 32 + ql] = v2f{m_ref, l_tot};
  barrier_lds_only();
  if (q >= args.nq_valid) return;
  v2f mls[NS];
  float m = -INFINITY;
#pragma unroll
  for (int s = 0; s < NS; s++) {
    mls[s] = ml[(qw * NS + s) * 32 + ql];
    m = fmaxf(m, mls[s][0]);
  }
  float l = 0.f, wgt[NS];
#pragma unroll
  for (int s = 0; s < NS; s++) {
    wgt[s] = __builtin_amdgcn_exp2f(mls[s][0] - m);            // 0 for a split that saw no tile
    l = __builtin_fmaf(mls[s][1], wgt[s], l);
  }
  const float inv_l = 1.0f / l;
  unsigned short* Oh = args.O + args.oview.row(bh, q);
#pragma unroll
  for (int cb = 0; cb < KS; cb++)
    if (cb % NS == g) {
#pragma unroll
      for (int aa = 0; aa < 4; aa++) {
        v4f o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < NS; s++) {
          v4f x;
          if (s == g) x = v4f{oacc[cb][4 * aa], oacc[cb][4 * aa + 1], oacc[cb][4 * aa + 2], oacc[cb][4 * aa + 3]};
          else x = *(const v4f*)(xch + ((((qw * NS + s) * KS + cb) * 4 + aa) * 64 + lane) * 4);
#pragma unroll
          for (int e = 0; e < 4; e++) o[e] = __builtin_fmaf(x[e], wgt[s], o[e]);
        }
        v4us ob;
#pragma unroll
        for (int e = 0; e < 4; e++) ob[e] = float_to_bf16_bits(o[e] * inv_l);
        *(v4us*)(Oh + 32 * cb + 8 * aa + 4 * h) = ob;
      }
    }
  if (g == 0 && h == 0) args.LSE[(size_t)bh * args.nq_valid + q] = (m + __builtin_amdgcn_logf(l) - kLog2_127) * kLn2;
}

}  // namespace sage
