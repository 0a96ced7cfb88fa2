// Fused INT8 attention backward (paper Algorithm 2) for gfx950.
//
// sage_bwd_kernel: a workgroup of 8 waves owns two adjacent KV blocks (one per group of 4
// waves) and walks the Q blocks i from the last one down.  The operands of the coming Q blocks
// are copied global -> LDS asynchronously (LDS-DMA loads) into double buffers.  Per (i, j) tile
// and group there are three phases:
//   phase A  each wave takes one 32x32 quadrant (qb, kb) of the tile:
//            S = Q^ K^^T on INT8 MFMA, dP = dO V^T on bf16 MFMA (the one unquantised matmul),
//            P = exp(S - L), dS = P o (dP - delta), kept in registers; the wave maxima of P and
//            |dS| go to LDS.
//   phase Q  with the tile-wide maxima: psi(P), psi(dS) to LDS as MFMA operand fragments, and
//            the psi(dS) fragments also to the scratch buffer (the dQ kernel transposes them).
//   phase B  each wave takes one 32-channel slice of the outputs and contracts over the whole
//            tile: dV^T += dO^^T P^, dK^T += Q^^T dS^ (accumulated in FP32 registers with the
//            per-tile scales).
// The phases are software-pipelined over ONE workgroup barrier per tile (see the kernel).
// sage_bwd_single_kernel and sage_bwd_wide_kernel divide the same arithmetic over the waves in other ways, for calls with few KV
// blocks and with many.
// A second kernel (sage_bwd_dq_kernel) owns two Q blocks per workgroup and forms
//   dQ_i = sum_j s_dS(i,j) s_K(j) sm_scale * (dS^_ij K^_j)
// from the stored INT8 tiles: a plain scaled INT8 GEMM with no atomics, so dQ is
// deterministic.  It is bound by the memory pipeline (the tiles are read once, from HBM), so
// its work goes into how the copies are issued and how dQ leaves, not into its arithmetic.
// (A first version added dQ with FP32 atomics from the first kernel; at N=8192 the 4.3e9
// atomic adds alone took 13 ms.)
//
// S is formed untransposed (queries x keys): an accumulator lane then holds one key and 16
// queries, which is the B-operand form of the two contractions over queries (dV, dK).  The
// contraction over keys (dQ) needs dS^ with one query per lane; scattering it bytewise through
// LDS cost more LDS time than all operand reads together, hence a transposing MFMA (one matrix
// instruction against a permutation matrix), which runs in the dQ kernel: that kernel waits for
// memory and has the issue slots to spare, this one does not.
#pragma once

#include <type_traits>

#include "common.h"

namespace sage {

struct BwdArgs {
  const int8_t* QF;    // F layout   (S recompute, A operand)
  const int8_t* QT;    // TF layout  (dK, A operand)
  const int8_t* KF;    // F layout   (S recompute, B operand)
  const int8_t* dOT;   // TF layout  (dV, A operand)
  const unsigned short* V;    // bf16, rows addressed through `cv` (dense [BH, N, D] or the caller's token-major tensors)
  const unsigned short* dO;   // bf16, likewise
  RowView cv;                 // rows of the K-like tensors V, dK, dV
  RowView cvq;                // rows of the Q-like tensor dO
  const float* sQ;
  const float* sK;
  const float* sdO;
  const float* nL2;    // [BH, N]  -LSE * log2(e)
  const float* delta;  // [BH, N]  -rowsum(dO o O)
  const float* bias;   // Q-smoothing logit bias [BH, N/64, N] (log2 domain) or nullptr
  const float* muQ;    // Q-smoothing block means [BH, N/64, D] or nullptr
  int8_t* dSq;         // psi(dS) tiles [heads, N/64, ds_pitch, 4096]: the four quadrant fragments as phase Q forms them
  int ds_pitch;        // tiles per Q-block row of that array (>= N/64)
  float* sdS;          // their scales [heads, N/64, ds_pitch]
  int stream_ds;       // the tiles are stored past the caches (see ds_traffic)
  float* tmax;         // B_q = 128: (max P, max |dS|) of the tiles of the even Q blocks [heads, N/64, ds_pitch][2], see MODE
  int bh0;             // first head of this launch (the scratch above is indexed from it)
  unsigned short* dK;  // bf16 [BH, N, D]
  unsigned short* dV;
  int BH, N;           // N = rows of the K-like workspace tensors (N_kv rounded up to a multiple of 64)
  int nvalid;          // keys >= nvalid do not exist (nvalid = N unless N_kv is not a multiple of 64)
  int Nq;              // rows of the Q-like workspace tensors (N_q rounded up to a multiple of 64)
  int nq_valid;        // query rows >= nq_valid do not exist
  int shift_blocks;    // causal: Q block i sees KV blocks j <= i + shift_blocks ((N_kv - N_q) / 64), diagonal at equality
  int head_set;        // heads per XCD whose work items are interleaved (see work_item)
  int fold_end;        // order of the first workgroups (see folded)
  float sm_scale;
  float scale_log2e;
};

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kRoundMagic = 12582912.0f;   // 1.5 * 2^23: x + magic has rne(x) in its low mantissa bits
constexpr int kMagicBits = 0x4B400000;       // its bit pattern

template <int D>
struct BwdStageA {            // operands of phase A for one Q block
  int8_t qf[64 * D];          // Q^  F fragments
  int8_t dof[128 * D];        // bf16 dO as A fragments (32-row block, 16-channel step), XOR-swizzled slots
  float nl2[64];              // -L * log2(e)
  float dl[64];               // -delta
  float bias[128];            // Q-smoothing logit bias of this Q block for the workgroup's 128 keys
  float sc[64];               // s_Q[i] in every entry
};
template <int D>
struct BwdStageB {            // operands of phase B for one Q block
  int8_t qt[64 * D];          // Q^  TF fragments
  int8_t dot[64 * D];         // dO^ TF fragments
  float muq[D];               // Q-smoothing block mean
  float sc[64];               // s_Q[i] in the even entries, s_dO[i] in the odd ones
};
struct BwdExchange {          // per group of 4 waves and tile parity
  int8_t pb[4096];            // psi(P)  B fragments (q step, key block)
  int8_t dsb[4096];           // psi(dS) B fragments
};

// phase A element-wise work of one quadrant (`dp` holds dP - delta); MASK = some entries of the tile are masked: query row
// qrow0 + 8 aa + b of the tile sees key column kcol only up to column klim_row (the row itself on
// the causal diagonal, 63 elsewhere) and only if the key exists (kcol < kvalid)
template <bool MASK, bool QSMOOTH>
__device__ __forceinline__ void bwd_quadrant(const v16i& sacc, const v16f& dp, const float* __restrict__ nl2, const float c, const float bias_l,
                                             const int qrow0, const int kcol, const bool diag, const int kvalid,
                                             float (&p)[16], float (&ds)[16], float& pm, float& dm, float& cs) {
  float pm2[2] = {0.f, 0.f}, dm2[2] = {0.f, 0.f};
  cs = 0.f;
#pragma unroll
  for (int aa = 0; aa < 4; aa++) {
    const v4f l4 = *(const v4f*)(nl2 + 8 * aa);
#pragma unroll
    for (int b = 0; b < 4; b++) {
      const int r = 4 * aa + b;
      const float off = QSMOOTH ? bias_l + l4[b] : l4[b];
      float pv = __builtin_amdgcn_exp2f(__builtin_fmaf((float)sacc[r], c, off));
      if constexpr (MASK) pv = ((diag && (qrow0 + 8 * aa + b) < kcol) || kcol >= kvalid) ? 0.f : pv;
      const float dsv = pv * dp[r];
      p[r] = pv;
      ds[r] = dsv;
      pm2[aa & 1] = fmaxf(pm2[aa & 1], pv);
      dm2[aa & 1] = fmaxf(dm2[aa & 1], fabsf(dsv));
      if constexpr (QSMOOTH) cs += dsv;
    }
  }
  pm = fmaxf(pm2[0], pm2[1]);
  dm = fmaxf(dm2[0], dm2[1]);
}

// Q-smoothing: dK_bias = (dS^T 1) mu_Q^T with the unquantised column sums of a tile, on the FP32 matrix instruction (contraction
// over two) straight into the accumulators of dK, before the tile's own products are added: rows = channels, one key per lane, the two
// lane halves' sums are the two terms: `cs` = (this lane half's sum over the first 32 rows of the Q block + over the second) * sm_scale.
// (As 16 FMAs into accumulators of their own it took 16 more registers per 32 x 32 block of dK and a read of mu_Q per four channels.)
__device__ __forceinline__ v16f add_dk_bias(const v16f& dk, const float muq, const float cs) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(muq, cs, dk, 0, 0, 0);
}

// Schedule.  The tiles of a group (Q blocks i = nblk-1 .. i_first against its KV block) go
// through three phases,
//   A  S = Q^K^^T (INT8), dP = dO V^T (bf16), P, dS in registers, wave maxima to LDS,
//   Q  psi(P), psi(dS) with the tile maxima -> LDS operand fragments,
//   B  dV^T += dO^^T P^, dK^T += Q^^T dS^ (INT8) with FP32 accumulation,
// software-pipelined over the workgroup's ONE barrier per tile: interval t runs Q of tile t-1,
// A of tile t and B of tile t-2, so every phase finds its cross-wave inputs complete and the
// matrix work of one tile runs under the vector work of its neighbours.
//
// MODE.  psi(P) and psi(dS) share one scale per numerics block of B_q queries x B_kv keys (Algorithm 2 lines
// 6 and 9).  With B_q = 64 (kBwdFused) the block lies inside one interval of this kernel and the maxima come
// from the interval's own phase A.  With B_q = 128 a block spans two consecutive Q blocks (2m + 1, which the
// walk meets first, and 2m), one interval apart, with no registers or LDS left to hold a tile back.  The tile
// of Q block 2m finds its partner's maxima in the previous interval's; the tile of 2m + 1 needs maxima the
// walk has not reached.  So the kernel runs twice: kBwdMaxOnly visits the EVEN Q blocks only, does phase A
// alone and stores each tile's two maxima to args.tmax; kBwdPairedRows is the full kernel, whose phase Q
// combines its own maxima with the stored ones of the tile below (odd Q blocks; staged into LDS one interval
// ahead) or with the previous interval's (even Q blocks).  P and dS are recomputed bit for bit, so the maxima
// are exactly those of the values quantised.
constexpr int kBwdFused = 0, kBwdMaxOnly = 1, kBwdPairedRows = 2;

// KV128: numerics blocks of 128 keys.  In that direction the block is the two tiles the workgroup's
// two groups hold in the same interval, so phase Q takes the maxima over both groups' phase A (a group whose
// tile does not exist in an interval, above the diagonal or past the last KV block, contributes zeros); 64 x 128
// blocks therefore need one sweep only.
template <int D, bool CAUSAL, bool QSMOOTH, int MODE = kBwdFused, bool KV128 = false>
__global__ void __launch_bounds__(512, MODE == kBwdMaxOnly ? 4 : 1) sage_bwd_kernel(BwdArgs args) {
  // kBwdMaxOnly has no accumulators and no phase B: V stays in registers, the buffers of phase B go, and two workgroups
  // share a CU (52 KB of LDS, 128 registers)
  constexpr bool VREG = MODE == kBwdMaxOnly;
  constexpr int ISTEP = MODE == kBwdMaxOnly ? 2 : 1;     // Q blocks between two tiles of the walk
  constexpr int KS = D / 32;     // INT8 k-steps over d; channel blocks
  constexpr int KB = D / 16;     // bf16 k-steps over d
  constexpr int NPB = KS / 2;    // 32-row blocks per wave in phase B (2 for D=128, 1 for D=64)
  constexpr int TILE = 64 * D;   // bytes of one INT8 tile
  constexpr int NF = TILE / 1024;  // 1 KiB fragments per INT8 tile

  // One LDS object: with several, the compiler tags every LDS access with the variable it touches and
  // then makes reads of buffers that no asynchronous copy ever writes wait for all copies in flight.
  struct Lds {
    BwdStageA<D> stA[2];
    __attribute__((aligned(16))) int8_t stB_bytes[VREG ? 16 : 2 * sizeof(BwdStageB<D>)];
    __attribute__((aligned(16))) int8_t xch_bytes[VREG ? 16 : 4 * sizeof(BwdExchange)];   // [group][tile parity]
    int8_t vst[VREG ? 1 : 2][VREG ? 16 : 2 * D * 64];   // [group]: bf16 V_j as B fragments (key block, 16-channel step)
    unsigned red[2][2][4][2];                       // [group][tile parity][wave][max P, max |dS|] as bit patterns
    float csum[QSMOOTH ? 2 * 3 * 2 * 2 * 64 : 1];   // [group][tile % 3][q half][lane half][key]: column sums of dS
    float tmx[MODE == kBwdPairedRows ? 2 * 2 * 64 : 1];   // [tile parity][group][even lanes: max P, odd lanes: max |dS|]
  };
  __shared__ __attribute__((aligned(16))) Lds L;
  auto& stA = L.stA;
  auto& stB = *(BwdStageB<D>(*)[2])L.stB_bytes;
  auto& xch = *(BwdExchange(*)[2][2])L.xch_bytes;
  auto& vst = L.vst;
  auto& red = L.red;
  auto& csum = L.csum;
  auto& tmx = L.tmx;

  const int gidx = blockIdx.x;
  const int N = args.N;
  const int nblk = N / kBlock;        // KV blocks
  const int nqblk = args.Nq / kBlock; // Q blocks
  const int sb = CAUSAL ? args.shift_blocks : 0;
  const int npair = (nblk + 1) / 2;
  const WorkItem wi = work_item(MODE == kBwdMaxOnly ? folded(gidx, args.fold_end) : gidx, npair, args.head_set);
  const int hl = wi.head;             // head within this launch
  const int bh = args.bh0 + hl;
  const int jp = wi.item;             // small jp = most Q blocks under the causal mask: scheduled first

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = wave >> 2, w4 = wave & 3, gtid = tid & 255;
  const int ll = lane & 31, h = lane >> 5;
  const int qb = w4 >> 1, kb = w4 & 1;                     // phase A quadrant
  const int cb = (D == 128) ? w4 : (w4 & 1);               // phase B channel block
  const int blk0 = (D == 128) ? 0 : (w4 >> 1);             // phase B first 32-row block
  const int j = 2 * jp + grp;
  const bool gvalid = j < nblk;
  const int jc = gvalid ? j : nblk - 1;                    // clamped: an idle group still loads in bounds
  const int kvalid = min(64, args.nvalid - 64 * jc);       // key columns of this group's KV block that exist

  const size_t head = (size_t)bh * N * D;                  // in the dense K-like workspace tensors
  const size_t qhead = (size_t)bh * args.Nq * D;           // in the Q-like ones
  const size_t chead = args.cv.row(bh, 0);                 // in V, dK, dV
  const size_t rs = args.cv.row_stride;
  const size_t cqhead = args.cvq.row(bh, 0);               // in dO
  const size_t rsq = args.cvq.row_stride;
  const float sKj = args.sK[(size_t)bh * nblk + jc];

  // ---- operands that stay in registers for the whole loop ----
  v4i kfr[KS];
  {
    const int8_t* p = args.KF + head + ((size_t)(2 * jc + kb) * KS) * 1024 + lane * 16;
#pragma unroll
    for (int s = 0; s < KS; s++) kfr[s] = *(const v4i*)(p + s * 1024);
  }
  // bf16 V_j (B operand of dP): staged once in LDS as 1 KiB fragments (key block kb, 16-channel
  // step s), lane (key, half) holding V[key][16 s + 8 half .. + 8]; 16 fragments (d = 128) dealt
  // to the group's 4 waves.  Keeping it in registers instead would cost 32 of them, which the
  // prefetch of the streamed operands needs more.
  v8bf vreg[VREG ? KB : 1];
  if constexpr (VREG) {
    const unsigned short* pv = args.V + chead + (size_t)min(64 * jc + 32 * kb + ll, args.nvalid - 1) * rs + 8 * h;
#pragma unroll
    for (int s = 0; s < KB; s++) vreg[s] = *(const v8bf*)(pv + 16 * s);
  }
#pragma unroll
  for (int k = 0; k < (VREG ? 0 : (2 * KB + 3) / 4); k++) {
    const int f = w4 + 4 * k;
    if (f < 2 * KB) {
      const int fkb = f / KB, fs = f % KB;
      // (a key row that does not exist re-reads the last one that does: its P is masked to zero)
      const int vrow = min(64 * jc + 32 * fkb + ll, args.nvalid - 1);
      async_copy_16(args.V + chead + (size_t)vrow * rs + 16 * fs + 8 * h, vst[grp] + f * 1024);
    }
  }

  v16f dvacc[NPB], dkacc[NPB];
#pragma unroll
  for (int t = 0; t < NPB; t++)
#pragma unroll
    for (int r = 0; r < 16; r++) {
      dvacc[t][r] = 0.f;
      dkacc[t][r] = 0.f;
    }

  const int i_first = CAUSAL ? max(2 * jp - sb, 0) : 0;
  // tile t of this workgroup is Q block itop - ISTEP * t, down to i_first (kBwdMaxOnly: the even blocks only)
  const int itop = MODE == kBwdMaxOnly ? ((nqblk - 1) & ~1) : nqblk - 1;
  const int T = itop >= i_first ? (itop - i_first) / ISTEP + 1 : 0;
  // Asynchronous staging (global -> LDS, no registers) of the phase-A operands of Q block i.
  // Written without branches where the fragment counts divide evenly among the 8 waves (d = 128):
  // which array a wave copies from is a compile-time fact per copy, and the small vectors are
  // copied by every wave (duplicates of identical data), so that the steady-state interval stays
  // one basic block.  Every address is a wave-uniform base plus a 32-bit lane offset.
  // (LAST: Q block i may be the partial last block; query rows that do not exist re-read the last one
  // that does: their P is zero because the pre-pass gave them -L = -inf)
  auto load_A = [&](int i, BwdStageA<D>& st, auto last_tag) {
    constexpr bool LAST = decltype(last_tag)::value;
    const size_t toff = qhead + (size_t)i * TILE;
    const unsigned lane16 = lane * 16;
#pragma unroll
    for (int k = 0; k < (3 * NF + 7) / 8; k++) {
      const int o = wave + 8 * k;            // wave-uniform
      const bool all_q = 8 * k + 7 < NF, none_q = 8 * k >= NF;       // compile-time when NF % 8 == 0
      const bool in_range = 8 * k + 7 < 3 * NF || o < 3 * NF;
      if (all_q || (!none_q && o < NF)) {
        async_copy_16(args.QF + toff + o * 1024 + lane16, st.qf + o * 1024);
      } else if (in_range) {
        // bf16 dO fragment f = (32-row block, 16-channel step s); LDS slot l holds the piece of
        // (row, channel half) = (l ^ (s & 7)) so that the A-operand reads stay conflict-free
        const int f = o - NF;
        const int rb = f / KB, sst = f % KB;
        const unsigned orig = lane ^ (sst & 7);
        if constexpr (LAST) {
          const int row = min(64 * i + 32 * rb + (int)(orig & 31), args.nq_valid - 1);
          async_copy_16(args.dO + cqhead + (size_t)row * rsq + 16 * sst + 8 * (orig >> 5), st.dof + f * 1024);
        } else {
          const size_t loff = (orig & 31) * (2 * rsq) + (orig >> 5) * 16;          // bytes: row, channel half
          const char* base = (const char*)(args.dO + cqhead + (size_t)(64 * i + 32 * rb) * rsq + 16 * sst);
          async_copy_16(base + loff, st.dof + f * 1024);
        }
      }
    }
    // -L*log2e (even waves) or delta (odd waves), and s_Q[i] broadcast to 64 entries
    const float* vsrc = ((wave & 1) ? args.delta : args.nL2) + (size_t)bh * args.Nq + 64 * i;
    async_copy_4((const char*)vsrc + lane * 4, (wave & 1) ? st.dl : st.nl2);
    async_copy_4(args.sQ + (size_t)bh * nqblk + i, st.sc);
    if constexpr (QSMOOTH) {
      const char* brow = (const char*)(args.bias + ((size_t)bh * nqblk + i) * N + 128 * jp);
      if (wave == 5) async_copy_4(brow + lane * 4, st.bias);
      if (wave == 6 && 2 * jp + 1 < nblk) async_copy_4(brow + 256 + lane * 4, st.bias + 64);
    }
  };
  // ... and of its phase-B operands.
  auto load_B = [&](int i, BwdStageB<D>& st) {
    const size_t toff = qhead + (size_t)i * TILE;
    const unsigned lane16 = lane * 16;
#pragma unroll
    for (int k = 0; k < (2 * NF + 7) / 8; k++) {
      const int o = wave + 8 * k;
      const bool all_q = 8 * k + 7 < NF, none_q = 8 * k >= NF;
      const bool in_range = 8 * k + 7 < 2 * NF || o < 2 * NF;
      if (all_q || (!none_q && o < NF)) async_copy_16(args.QT + toff + o * 1024 + lane16, st.qt + o * 1024);
      else if (in_range) async_copy_16(args.dOT + toff + (o - NF) * 1024 + lane16, st.dot + (o - NF) * 1024);
    }
    // s_Q[i] (even lanes) and s_dO[i] (odd lanes)
    async_copy_4(((lane & 1) ? args.sdO : args.sQ) + (size_t)bh * nqblk + i, st.sc);
    if constexpr (QSMOOTH) {
      const char* mq = (const char*)(args.muQ + ((size_t)bh * nqblk + i) * D);
      if (wave == 3) async_copy_4(mq + lane * 4, st.muq);
      if (D == 128 && wave == 4) async_copy_4(mq + 256 + lane * 4, st.muq + 64);
    }
  };

  load_A(itop, stA[0], std::true_type{});
  barrier_all_memory();

  float p[16], ds[16];           // P and dS of the tile between its phases A and Q
  float sP_q = 0.f, sS_q = 0.f;  // tile scales found by the last phase Q
  unsigned prev_p = 0u, prev_d = 0u;   // kBwdPairedRows: the maxima (bit patterns) of the tile the last phase Q handled
  // One interval.  STEADY = all three phases are active and tile t is not on the diagonal: the
  // body is then free of branches, one basic block in which the compiler interleaves the three
  // independent phases (the LDS and MFMA latencies of one hide under the vector work of the others).
  auto interval = [&](const int t, auto steady_tag, auto b_before_a_tag) __attribute__((always_inline)) {
    constexpr bool STEADY = decltype(steady_tag)::value;
    constexpr bool B_BEFORE_A = decltype(b_before_a_tag)::value;
    const float sP_b = sP_q, sS_b = sS_q;      // scales of tile t - 2 (its phase Q ran in the last interval)
    const int ib = itop - ISTEP * (t - 2);     // Q blocks of the three tiles in flight
    const int iq = itop - ISTEP * (t - 1);
    const int ia = itop - ISTEP * t;
    const bool act_b = MODE != kBwdMaxOnly && (STEADY || (t >= 2 && gvalid && (!CAUSAL || ib + sb >= j)));
    const bool act_q = STEADY || (t >= 1 && t - 1 < T && gvalid && (!CAUSAL || iq + sb >= j));
    const bool act_a = STEADY || (t < T && gvalid && (!CAUSAL || ia + sb >= j));

    auto phase_b = [&]() __attribute__((always_inline)) {
    // ---------------- phase B of tile t - 2: channel block cb ----------------
    if (act_b) {
      const BwdStageB<D>& st = stB[t & 1];
      const BwdExchange& X = xch[grp][t & 1];
      const float w_dv = sP_b * st.sc[1];
      const float w_dk = sS_b * st.sc[0] * args.sm_scale;
#pragma unroll
      for (int tt = 0; tt < NPB; tt++) {
        const int kbo = blk0 + tt;
        if constexpr (QSMOOTH) {
          const float* cs = csum + ((grp * 3 + (t - 2) % 3) * 4 + h) * 64 + 32 * kbo + ll;
          dkacc[tt] = add_dk_bias(dkacc[tt], st.muq[32 * cb + ll], (cs[0] + cs[128]) * args.sm_scale);
        }
        v16i av, ak;
#pragma unroll
        for (int r = 0; r < 16; r++) {
          av[r] = 0;
          ak[r] = 0;
        }
#pragma unroll
        for (int qs = 0; qs < 2; qs++) {
          const v4i a1 = *(const v4i*)(st.dot + ((qs * KS + cb) * 64 + lane) * 16);
          const v4i b1 = *(const v4i*)(X.pb + ((qs * 2 + kbo) * 64 + lane) * 16);
          av = __builtin_amdgcn_mfma_i32_32x32x32_i8(a1, b1, av, 0, 0, 0);
          const v4i a2 = *(const v4i*)(st.qt + ((qs * KS + cb) * 64 + lane) * 16);
          const v4i b2 = *(const v4i*)(X.dsb + ((qs * 2 + kbo) * 64 + lane) * 16);
          ak = __builtin_amdgcn_mfma_i32_32x32x32_i8(a2, b2, ak, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 16; r++) {
          dvacc[tt][r] = __builtin_fmaf((float)av[r], w_dv, dvacc[tt][r]);
          dkacc[tt][r] = __builtin_fmaf((float)ak[r], w_dk, dkacc[tt][r]);
        }
      }
    }
    };
    // operands of the coming intervals; the copies are issued in two batches so that the eight
    // waves do not queue up behind each other at the memory pipeline
    if (STEADY || t + 1 < T) load_A(ia - ISTEP, stA[(t + 1) & 1], std::false_type{});

    __builtin_amdgcn_sched_barrier(0);
    // ---------------- phase Q of tile t - 1 ----------------
    if (act_q) {
      BwdExchange& X = xch[grp][(t - 1) & 1];
      // (the maxima are non-negative floats: they order like their bit patterns, and integer maxima
      // need no NaN canonicalisation of the loaded values)
      const unsigned(&R)[4][2] = red[grp][(t - 1) & 1];
      unsigned pu = max(max(R[0][0], R[1][0]), max(R[2][0], R[3][0]));
      unsigned du = max(max(R[0][1], R[1][1]), max(R[2][1], R[3][1]));
      if constexpr (KV128) {
        const unsigned(&R2)[4][2] = red[grp ^ 1][(t - 1) & 1];
        pu = max(pu, max(max(R2[0][0], R2[1][0]), max(R2[2][0], R2[3][0])));
        du = max(du, max(max(R2[0][1], R2[1][1]), max(R2[2][1], R2[3][1])));
      }
      if constexpr (MODE == kBwdPairedRows) {
        // the other Q block of the numerics block: below (iq odd: the stored maxima of tile (iq - 1, j), and of
        // its neighbour in the 128-key block, where those tiles exist) or above (iq even: the last interval's)
        const unsigned own_p = pu, own_d = du;
        if (iq & 1) {
          const unsigned* tm = (const unsigned*)(tmx + (((t - 1) & 1) * 2 + grp) * 64);
          if constexpr (KV128) {
            const int j0 = j & ~1;
            if (!CAUSAL || j0 <= iq - 1 + sb) {
              pu = max(pu, tm[0]);
              du = max(du, tm[1]);
            }
            if (j0 + 1 < nblk && (!CAUSAL || j0 + 1 <= iq - 1 + sb)) {
              pu = max(pu, tm[2]);
              du = max(du, tm[3]);
            }
          } else if (!CAUSAL || j <= iq - 1 + sb) {
            pu = max(pu, tm[0]);
            du = max(du, tm[1]);
          }
        } else if (iq + 1 < nqblk) {
          pu = max(pu, prev_p);
          du = max(du, prev_d);
        }
        prev_p = own_p;
        prev_d = own_d;
      }
      const float pm = __uint_as_float(pu), dm = __uint_as_float(du);
      if constexpr (MODE == kBwdMaxOnly) {
        // this tile's two maxima, for the pass over the numerics blocks; nothing is quantised in this mode
        if (w4 == 0 && lane == 0) {
          const size_t tile = ((size_t)hl * nqblk + iq) * args.ds_pitch + j;
          *(v2f*)(args.tmax + 2 * tile) = v2f{pm, dm};
        }
      } else {
      // the per-tile scales of P and dS are internal (never stored bit-exactly): 127/a via rcp
      const float rP = pm > 0.f ? 127.0f * __builtin_amdgcn_rcpf(pm) : 0.f;
      const float rS = dm > 0.f ? 127.0f * __builtin_amdgcn_rcpf(dm) : 0.f;
      sP_q = pm * (1.0f / 127.0f);
      sS_q = dm * (1.0f / 127.0f);
      v4i pf, df;
#pragma unroll
      for (int aa = 0; aa < 4; aa++) {
        unsigned ub[4];
#pragma unroll
        for (int b = 0; b < 4; b++) ub[b] = __float_as_uint(__builtin_fmaf(ds[4 * aa + b], rS, kRoundMagic));
        const unsigned lo = __builtin_amdgcn_perm(ub[1], ub[0], 0x0c0c0400u);
        const unsigned hi = __builtin_amdgcn_perm(ub[3], ub[2], 0x04000c0cu);
        df[aa] = (int)(lo | hi);
      }
#pragma unroll
      for (int aa = 0; aa < 4; aa++) {
        unsigned up = 0;
#pragma unroll
        for (int b = 0; b < 4; b++) up = __builtin_amdgcn_cvt_pk_u8_f32(p[4 * aa + b] * rP, b, up);
        pf[aa] = (int)up;
      }
      *(v4i*)(X.pb + ((qb * 2 + kb) * 64 + lane) * 16) = pf;
      *(v4i*)(X.dsb + ((qb * 2 + kb) * 64 + lane) * 16) = df;
      {
        // the same fragment goes to the scratch buffer for the dQ kernel: fragment (qb, kb), lane (key, h),
        // byte 4 a + b = psi(dS)[32 qb + 8 a + 4 h + b][32 kb + key]
        // (tiles and scales share one index: a second index product costs the Q-smoothing instantiation a spill)
        const size_t tile = ((size_t)hl * nqblk + iq) * args.ds_pitch + j;
        *(v4i*)(args.dSq + tile * 4096 + ((qb * 2 + kb) * 64 + lane) * 16) = df;
        args.sdS[tile] = sS_q;   // the same value from every lane: no branch
      }
      }
    }
    if constexpr (MODE != kBwdMaxOnly) {
      if (STEADY || (t >= 1 && t - 1 < T)) load_B(iq, stB[(t - 1) & 1]);
    }
    if constexpr (MODE == kBwdPairedRows) {
      // tile t has its phase Q in the next interval: if its Q block is odd, the stored maxima of the tile below
      // it (and, with 128-key blocks, of that tile's neighbour: entries j0 and j0 + 1 are adjacent; the rows of
      // the table are three entries longer than a row of tiles).  Each wave copies its group's two or four
      // floats: lanes 0, 1 (, 2, 3) = max P, max |dS| (, of the neighbour); the other lanes repeat them.
      if ((STEADY || t < T) && (ia & 1)) {
        const size_t tile = ((size_t)hl * nqblk + ia - 1) * args.ds_pitch + (KV128 ? (jc & ~1) : jc);
        async_copy_4(args.tmax + 2 * tile + (lane & (KV128 ? 3 : 1)), tmx + ((t & 1) * 2 + grp) * 64);
      }
    }

    __builtin_amdgcn_sched_barrier(0);
    if constexpr (B_BEFORE_A) {
      phase_b();
      __builtin_amdgcn_sched_barrier(0);
    }
    // The two waves of a SIMD are wave w (first group) and w + 4 (second group); the arbiter favours the
    // older one, which then idles at the interval's barrier.  Raising the younger wave's priority for
    // its MFMA-dense phase evens the two out (measured: 2-3 % of the kernel).
    if (STEADY && grp == 1) __builtin_amdgcn_s_setprio(1);
    // ---------------- phase A of tile t: quadrant (qb, kb) ----------------
    if (act_a) {
      const BwdStageA<D>& st = stA[t & 1];
      // The two MFMA chains (S over INT8 steps, dP over bf16 steps) are interleaved, and the LDS
      // reads of their operands run two bf16 steps ahead of the MFMAs that consume them.
      v4i qa[KS];
      v8bf da[KB], vb[KB];
      const int8_t* qfp = st.qf + (qb * KS * 64 + lane) * 16;
      const int8_t* vbp = vst[VREG ? 0 : grp] + (kb * KB * 64 + lane) * 16;
      auto ld = [&](int s) {
        if (s % 2 == 0) qa[s / 2] = *(const v4i*)(qfp + (s / 2) * 1024);
        da[s] = *(const v8bf*)(st.dof + ((qb * KB + s) * 64 + (lane ^ (s & 7))) * 16);
        if constexpr (VREG) vb[s] = vreg[s];
        else vb[s] = *(const v8bf*)(vbp + s * 1024);
      };
      ld(0);
      ld(1);
      v16i sacc;
      v16f dp;
      // dS = P o (dP - delta): the dP chain starts from -delta of the rows this lane's registers hold
      // (register 4a + b = query 8a + 4h + b of the quadrant), which saves the subtraction per entry.
      const float* dl = st.dl + 32 * qb + 4 * h;
#pragma unroll
      for (int aa = 0; aa < 4; aa++) {
        const v4f d4 = *(const v4f*)(dl + 8 * aa);
#pragma unroll
        for (int b = 0; b < 4; b++) dp[4 * aa + b] = d4[b];
      }
#pragma unroll
      for (int r = 0; r < 16; r++) sacc[r] = 0;
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int s = 0; s < KB; s++) {
        if (s + 2 < KB) ld(s + 2);
        if (s % 2 == 0) sacc = __builtin_amdgcn_mfma_i32_32x32x32_i8(qa[s / 2], kfr[s / 2], sacc, 0, 0, 0);
        dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(da[s], vb[s], dp, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
      const float c = st.sc[0] * sKj * args.scale_log2e;
      float bias_l = 0.f;
      if constexpr (QSMOOTH) bias_l = st.bias[64 * grp + 32 * kb + ll];
      const float* nl2 = st.nl2 + 32 * qb + 4 * h;
      float pm, dm, cs;
      if (!STEADY && ((CAUSAL && ia + sb == j) || kvalid < 64))
        bwd_quadrant<true, QSMOOTH>(sacc, dp, nl2, c, bias_l, 32 * qb + 4 * h, 32 * kb + ll, CAUSAL && ia + sb == j, kvalid,
                                    p, ds, pm, dm, cs);
      else
        bwd_quadrant<false, QSMOOTH>(sacc, dp, nl2, c, bias_l, 0, 0, false, 64, p, ds, pm, dm, cs);
      pm = wave_max_nonneg_f32(pm);
      dm = wave_max_nonneg_f32(dm);
      // every lane stores the same pair (one LDS write, no branch)
      red[grp][t & 1][w4][0] = __float_as_uint(pm);
      red[grp][t & 1][w4][1] = __float_as_uint(dm);
      if constexpr (QSMOOTH) csum[((grp * 3 + t % 3) * 4 + 2 * qb + h) * 64 + 32 * kb + ll] = cs;
    } else if constexpr (KV128) {
      // no tile for this group in this interval: nothing for the other group's block maxima
      red[grp][t & 1][w4][0] = 0u;
      red[grp][t & 1][w4][1] = 0u;
    }

    __builtin_amdgcn_sched_barrier(0);
    if (STEADY) __builtin_amdgcn_s_setprio(0);
    if constexpr (!B_BEFORE_A) phase_b();
    barrier_all_memory();   // the interval's LDS traffic, copies and stores are complete
  };
  // steady intervals: t >= DRAIN (the tiles of all phases exist), tile t above the diagonal and not the last row
  // (a KV block with keys that do not exist masks them in every tile: no branch-free intervals for its group)
  // (under the mask: while Q block itop - ISTEP * t lies above the group's diagonal block j - sb)
  const int t_steady_end = (!gvalid || kvalid < 64) ? 0 : (CAUSAL ? min((itop + sb - j + ISTEP - 1) / ISTEP, T - 1) : T - 1);
  int t = 0;
  constexpr int DRAIN = MODE == kBwdMaxOnly ? 1 : 2;       // phases behind A
  for (; t < DRAIN && t < T + DRAIN; t++) interval(t, std::false_type{}, std::false_type{});
  // (the second group's waves take phase B before phase A: the two waves of a SIMD then do not reach the
  // MFMA-dense phase at the same time)
  if (grp == 0) {
    for (; t < t_steady_end; t++) interval(t, std::true_type{}, std::false_type{});
  } else {
    for (; t < t_steady_end; t++) interval(t, std::true_type{}, std::true_type{});
  }
  for (; t < T + DRAIN; t++) interval(t, std::false_type{}, std::false_type{});

  if (!gvalid) return;

  // ---- write dV, dK (bf16) ----
#pragma unroll
  for (int t = 0; t < NPB; t++) {
    const int key = 64 * j + 32 * (blk0 + t) + ll;
    unsigned short* pv = args.dV + chead + (size_t)key * rs + 32 * cb + 4 * h;
    unsigned short* pk = args.dK + chead + (size_t)key * rs + 32 * cb + 4 * h;
#pragma unroll
    for (int aa = 0; aa < 4; aa++) {
      v4us ov, ok;
#pragma unroll
      for (int b = 0; b < 4; b++) {
        ov[b] = float_to_bf16_bits(dvacc[t][4 * aa + b]);
        ok[b] = float_to_bf16_bits(dkacc[t][4 * aa + b]);
      }
      if (key < args.nvalid) {
        *(v4us*)(pv + 8 * aa) = ov;
        *(v4us*)(pk + 8 * aa) = ok;
      }
    }
  }
}

// ---- one KV block per workgroup ------------------------------------------------------------------------
// sage_bwd_single_kernel (numerics blocks of 64 x 64).  The kernel above gives each group of four waves a KV block and all
// three phases; one of its intervals takes about 4850 cycles, and a call with few heads takes the time of one
// workgroup's chain of intervals.  Here the eight waves share ONE KV block and divide the phases: waves 0-3 ("front") run
// phases Q and A, waves 4-7 ("back") issue every copy and run phase B, so an interval takes about 2700 cycles for half as
// many tiles, and twice as many workgroups share the work.  Each SIMD has one wave of either kind.  The arithmetic of
// every value and its order are those of sage_bwd_kernel, so both give the same bits.
// Measured, backward kernel in us: 8 heads of N = 1000 d = 128: 43 -> 28; 4 heads of 4096: 131 -> 78; 32 heads of 2048: 89 -> 103
// (a full machine pays for staging the Q side once per KV block instead of once per two).  At d = 64 two of these workgroups
// fit a CU (120 registers, 81 KB of LDS), four waves to a SIMD: 64 heads of N = 8192: 1772 -> 1598.
//
// The front waves hold V in registers (no accumulators there), and the phases' operands come two intervals ahead in three
// stages each: a back wave waits for the copies of the interval before, and a front wave (whose only global memory
// operations are the stores of psi(dS)) for none.
template <int D>
struct BwdStageA1 {           // operands of phase A for one Q block
  int8_t qf[64 * D];          // Q^  F fragments
  int8_t dof[128 * D];        // bf16 dO as A fragments, XOR-swizzled slots (see BwdStageA)
  float nl2[64];              // -L * log2(e)
  float dl[64];               // -delta
  float bias[64];             // Q-smoothing logit bias of this Q block for the workgroup's 64 keys
};
template <int D>
struct BwdStageB1 {           // operands of phase B for one Q block
  int8_t qt[64 * D];          // Q^  TF fragments
  int8_t dot[64 * D];         // dO^ TF fragments
  float muq[D];               // Q-smoothing block mean
};


// Stage of the dQ kernels' loads: past the last one of a walk that one again (never used).  (Host code too, as below.)
__host__ __device__ inline int dq_stage(int j, int n_j) { return j < n_j ? j : n_j - 1; }

// The Q blocks such a workgroup walks, from the last one down: tile t = Q block itop - t, t = 0 .. T - 1.  Interval t
// copies the operands of phase A of tile t + 2 and of phase B of tile t, past the last tile that one again (never used):
// every interval issues the same copies, so that they can be counted.  (Host code too: a test goes through every index.)
struct SingleWalk {
  int itop, i_first, T;
  __host__ __device__ SingleWalk(int nqblk, int first) : itop(nqblk - 1), i_first(first), T(nqblk - first) {}
  __host__ __device__ int at(int t) const { return itop - t > i_first ? itop - t : i_first; }   // Q block of tile t
  // The partial last Q block is copied by the two first copies, which clamp each row (dO_row_clamped).  The copies inside
  // the loop do not clamp, and a walk of one tile would repeat that very block there: it repeats the block's first row.
  __host__ __device__ int loop_row_step() const { return T > 1 ? 1 : 0; }
};
// Row of dO that the copy of query row `row` reads: a row that does not exist re-reads the last one that does.
__host__ __device__ inline int dO_row_clamped(int row, int nq_valid) { return row < nq_valid ? row : nq_valid - 1; }

template <int D, bool CAUSAL, bool QSMOOTH>
__global__ void __launch_bounds__(512, 1) sage_bwd_single_kernel(BwdArgs args) {
  constexpr int KS = D / 32;     // INT8 k-steps over d; channel blocks
  constexpr int KB = D / 16;     // bf16 k-steps over d
  constexpr int NPB = KS / 2;    // 32-row blocks per wave in phase B
  constexpr int TILE = 64 * D;
  constexpr int NF = TILE / 1024;
  struct Lds {
    BwdStageA1<D> stA[3];
    BwdStageB1<D> stB[3];
    BwdExchange xch[2];                             // [tile parity]
    unsigned red[2][4][2];                          // [tile parity][wave][max P, max |dS|] as bit patterns
    float scl[2][2];                                // [tile parity][s_P, s_dS]
    float csum[QSMOOTH ? 3 * 2 * 2 * 64 : 1];       // [tile % 3][q half][lane half][key]: column sums of dS
  };
  __shared__ __attribute__((aligned(16))) Lds L;

  const int N = args.N;
  const int nblk = N / kBlock;        // KV blocks
  const int nqblk = args.Nq / kBlock; // Q blocks
  const int sb = CAUSAL ? args.shift_blocks : 0;
  const WorkItem wi = work_item(D == 64 && !QSMOOTH ? folded(blockIdx.x, args.fold_end) : blockIdx.x, nblk, args.head_set);
  const int hl = wi.head;
  const int bh = args.bh0 + hl;
  const int j = wi.item;              // small j = most Q blocks under the causal mask: scheduled first
  const int kvalid = min(64, args.nvalid - 64 * j);

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool front = wave < 4;
  const int w4 = wave & 3;
  const int ll = lane & 31, h = lane >> 5;
  const int qb = w4 >> 1, kb = w4 & 1;                     // phase A quadrant
  const int cb = (D == 128) ? w4 : (w4 & 1);               // phase B channel block
  const int blk0 = (D == 128) ? 0 : (w4 >> 1);             // phase B first 32-row block

  const size_t qhead = (size_t)bh * args.Nq * D;
  const size_t rs = args.cv.row_stride, rsq = args.cvq.row_stride;
  const size_t chead = args.cv.row(bh, 0), cqhead = args.cvq.row(bh, 0);
  const float* sQh = args.sQ + (size_t)bh * nqblk;
  const float* sdOh = args.sdO + (size_t)bh * nqblk;
  const SingleWalk walk(nqblk, CAUSAL ? max(j - sb, 0) : 0);   // (at least one tile: the diagonal)
  const int itop = walk.itop, i_first = walk.i_first, T = walk.T;
  const size_t rsq_loop = walk.loop_row_step() ? rsq : 0;

  // This wave's copies for Q block i (back waves): phase A's fragments are dealt to the four waves, then phase B's.
  auto copy_A = [&](int i, BwdStageA1<D>& st, auto last_tag) __attribute__((always_inline)) {
    constexpr bool LAST = decltype(last_tag)::value;       // Q block i may be the partial last one
    const size_t toff = qhead + (size_t)i * TILE;
#pragma unroll
    for (int k = 0; k < 3 * NF / 4; k++) {
      const int o = w4 + 4 * k;
      if (4 * k < NF) {
        async_copy_16(args.QF + toff + o * 1024 + lane * 16, st.qf + o * 1024);
      } else {
        const int f = o - NF;
        const int rb = f / KB, sst = f % KB;
        const unsigned orig = lane ^ (sst & 7);
        const int r = 32 * rb + (int)(orig & 31);
        const size_t row = LAST ? (size_t)dO_row_clamped(64 * i + r, args.nq_valid) * rsq : (size_t)(64 * i) * rsq + r * rsq_loop;
        async_copy_16(args.dO + cqhead + row + 16 * sst + 8 * (orig >> 5), st.dof + f * 1024);
      }
    }
    const float* vsrc = ((w4 & 1) ? args.delta : args.nL2) + (size_t)bh * args.Nq + 64 * i;
    async_copy_4(vsrc + lane, (w4 & 1) ? st.dl : st.nl2);
    if constexpr (QSMOOTH) async_copy_4(args.bias + ((size_t)bh * nqblk + i) * N + 64 * j + lane, st.bias);
  };
  auto copy_B = [&](int i, BwdStageB1<D>& st) __attribute__((always_inline)) {
    const size_t toff = qhead + (size_t)i * TILE;
#pragma unroll
    for (int k = 0; k < 2 * NF / 4; k++) {
      const int o = w4 + 4 * k;
      if (4 * k < NF) async_copy_16(args.QT + toff + o * 1024 + lane * 16, st.qt + o * 1024);
      else async_copy_16(args.dOT + toff + (o - NF) * 1024 + lane * 16, st.dot + (o - NF) * 1024);
    }
    if constexpr (QSMOOTH) {
      const int part = D == 128 ? (w4 & 1) * 64 : 0;
      async_copy_4(args.muQ + ((size_t)bh * nqblk + i) * D + part + lane, st.muq + part);
    }
  };
  constexpr int COPIES = 5 * NF / 4 + 1 + (QSMOOTH ? 2 : 0);   // per back wave and interval
  static_assert(NF % 4 == 0 && COPIES < 64, "fragments dealt evenly; vmcnt has six bits");

  if (!front) {
    copy_A(itop, L.stA[0], std::true_type{});
    copy_A(walk.at(1), L.stA[1], std::true_type{});
  }

  if (front) {
    // ================= front waves: phases Q and A, quadrant (qb, kb) =================
    __builtin_amdgcn_s_setprio(1);     // (the longer chain of the two; 2 to 5 % where workgroups share a CU)
    const float sKj = args.sK[(size_t)bh * nblk + j];
    v4i kfr[KS];
    v8bf vb[KB];
    {
      const int8_t* p = args.KF + (size_t)bh * N * D + ((size_t)(2 * j + kb) * KS) * 1024 + lane * 16;
#pragma unroll
      for (int s = 0; s < KS; s++) kfr[s] = *(const v4i*)(p + s * 1024);
      // (a key row that does not exist re-reads the last one that does: its P is masked to zero)
      const unsigned short* pv = args.V + chead + (size_t)min(64 * j + 32 * kb + ll, args.nvalid - 1) * rs + 8 * h;
#pragma unroll
      for (int s = 0; s < KB; s++) vb[s] = *(const v8bf*)(pv + 16 * s);
    }
    float p[16], ds[16];           // P and dS of the tile between its phases A and Q
    v4i qa[KS];
    v8bf da[KB];
    v16f dp;                       // starts from -delta, becomes dP - delta
    auto read_delta = [&](const int t) __attribute__((always_inline)) {
      const float* dl = L.stA[t % 3].dl + 32 * qb + 4 * h;
#pragma unroll
      for (int aa = 0; aa < 4; aa++) {
        const v4f d4 = *(const v4f*)(dl + 8 * aa);
#pragma unroll
        for (int b = 0; b < 4; b++) dp[4 * aa + b] = d4[b];
      }
    };
    auto read_A = [&](const int t) __attribute__((always_inline)) {
      const BwdStageA1<D>& st = L.stA[t % 3];
      // (with Q-smoothing a CU holds one of these workgroups whatever the registers: -delta is read ahead as well, 3 %; at d = 64
      // behind the operands, which the first products wait for: 16 heads of N = 2048 69.1 -> 68.4 us, 4 of 4096 107.3 -> 106.1, d =
      // 128 78.0 -> 79.6)
      if constexpr (QSMOOTH && D == 128) read_delta(t);
#pragma unroll
      for (int s = 0; s < KB; s++) {
        if (s % 2 == 0) qa[s / 2] = *(const v4i*)(st.qf + ((qb * KS + s / 2) * 64 + lane) * 16);
        da[s] = *(const v8bf*)(st.dof + ((qb * KB + s) * 64 + (lane ^ (s & 7))) * 16);
      }
      if constexpr (QSMOOTH && D == 64) read_delta(t);
    };
    auto phase_Q = [&](const int t) __attribute__((always_inline)) {   // tile t
      BwdExchange& X = L.xch[t & 1];
      const unsigned(&R)[4][2] = L.red[t & 1];
      const unsigned pu = max(max(R[0][0], R[1][0]), max(R[2][0], R[3][0]));
      const unsigned du = max(max(R[0][1], R[1][1]), max(R[2][1], R[3][1]));
      const float pm = __uint_as_float(pu), dm = __uint_as_float(du);
      const float rP = pm > 0.f ? 127.0f * __builtin_amdgcn_rcpf(pm) : 0.f;
      const float rS = dm > 0.f ? 127.0f * __builtin_amdgcn_rcpf(dm) : 0.f;
      const float sP = pm * (1.0f / 127.0f), sS = dm * (1.0f / 127.0f);
      v4i pf, df;
#pragma unroll
      for (int aa = 0; aa < 4; aa++) {
        unsigned ub[4];
#pragma unroll
        for (int b = 0; b < 4; b++) ub[b] = __float_as_uint(__builtin_fmaf(ds[4 * aa + b], rS, kRoundMagic));
        df[aa] = (int)(__builtin_amdgcn_perm(ub[1], ub[0], 0x0c0c0400u) | __builtin_amdgcn_perm(ub[3], ub[2], 0x04000c0cu));
      }
#pragma unroll
      for (int aa = 0; aa < 4; aa++) {
        unsigned up = 0;
#pragma unroll
        for (int b = 0; b < 4; b++) up = __builtin_amdgcn_cvt_pk_u8_f32(p[4 * aa + b] * rP, b, up);
        pf[aa] = (int)up;
      }
      *(v4i*)(X.pb + ((qb * 2 + kb) * 64 + lane) * 16) = pf;
      *(v4i*)(X.dsb + ((qb * 2 + kb) * 64 + lane) * 16) = df;
      L.scl[t & 1][0] = sP;        // (the same values from every lane)
      L.scl[t & 1][1] = sS;
      const size_t tile = ((size_t)hl * nqblk + (itop - t)) * args.ds_pitch + j;
      *(v4i*)(args.dSq + tile * 4096 + ((qb * 2 + kb) * 64 + lane) * 16) = df;
      args.sdS[tile] = sS;
    };
    // (the operands of the products, qa and da, have been read)
    auto phase_A = [&](const int t, const float sq, auto mask_tag) __attribute__((always_inline)) {
      constexpr bool MASK = decltype(mask_tag)::value;
      const BwdStageA1<D>& st = L.stA[t % 3];
      v16i sacc;
      if constexpr (!QSMOOTH) read_delta(t);
#pragma unroll
      for (int r = 0; r < 16; r++) sacc[r] = 0;
#pragma unroll
      for (int s = 0; s < KB; s++) {
        if (s % 2 == 0) sacc = __builtin_amdgcn_mfma_i32_32x32x32_i8(qa[s / 2], kfr[s / 2], sacc, 0, 0, 0);
        dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(da[s], vb[s], dp, 0, 0, 0);
      }
      const float c = sq * sKj * args.scale_log2e;
      float bias_l = 0.f;
      if constexpr (QSMOOTH) bias_l = st.bias[32 * kb + ll];
      const int ia = itop - t;
      float pm, dm, cs;
      if constexpr (MASK)
        bwd_quadrant<true, QSMOOTH>(sacc, dp, st.nl2 + 32 * qb + 4 * h, c, bias_l, 32 * qb + 4 * h, 32 * kb + ll, CAUSAL && ia + sb == j,
                                    kvalid, p, ds, pm, dm, cs);
      else
        bwd_quadrant<false, QSMOOTH>(sacc, dp, st.nl2 + 32 * qb + 4 * h, c, bias_l, 0, 0, false, 64, p, ds, pm, dm, cs);
      pm = wave_max_nonneg_f32(pm);
      dm = wave_max_nonneg_f32(dm);
      L.red[t & 1][w4][0] = __float_as_uint(pm);
      L.red[t & 1][w4][1] = __float_as_uint(dm);
      if constexpr (QSMOOTH) L.csum[((t % 3) * 4 + 2 * qb + h) * 64 + 32 * kb + ll] = cs;
    };
    barrier_all_memory();
    float sq = scalar_load(sQh + itop);
    // unmasked tiles: 0 .. t_plain - 1
    const int t_plain = kvalid < 64 ? 0 : (CAUSAL && i_first + sb == j ? T - 1 : T);
    for (int t = 0; t < T + 2; t++) {
      const float sqn = scalar_load(sQh + max(itop - t - 1, i_first));
      if (t >= 1 && t < t_plain) {
        read_A(t);
        phase_Q(t - 1);
        phase_A(t, sq, std::false_type{});
      } else {
        if (t >= 1 && t <= T) phase_Q(t - 1);
        if (t < T) {
          read_A(t);
          phase_A(t, sq, std::true_type{});      // (the masked form leaves unmasked entries as they are)
        }
      }
      sq = sqn;
      barrier_lds_only();
    }
    return;
  }

  // ================= back waves: the copies, phase B, channel block cb =================
  v16f dvacc[NPB], dkacc[NPB];
#pragma unroll
  for (int t = 0; t < NPB; t++)
#pragma unroll
    for (int r = 0; r < 16; r++) {
      dvacc[t][r] = 0.f;
      dkacc[t][r] = 0.f;
    }
  barrier_all_memory();
  float sq0 = 0.f, sd0 = 0.f, sq1 = 0.f, sd1 = 0.f;          // s_Q, s_dO of tiles t - 2 and t - 1
  for (int t = 0; t < T + 2; t++) {
    const int in = walk.at(t);
    // the terms of dK_bias of tile t - 2 are read ahead of the copies, whose issue takes longer than the reads
    float muq = 0.f, cs[NPB] = {};
    if (QSMOOTH && t >= 2) {
      muq = L.stB[(t - 2) % 3].muq[32 * cb + ll];
#pragma unroll
      for (int tt = 0; tt < NPB; tt++) {
        const float* c2 = L.csum + (((t - 2) % 3) * 4 + h) * 64 + 32 * (blk0 + tt) + ll;
        cs[tt] = (c2[0] + c2[128]) * args.sm_scale;
      }
    }
    copy_A(walk.at(t + 2), L.stA[(t + 2) % 3], std::false_type{});
    copy_B(in, L.stB[t % 3]);
    const float sqn = scalar_load(sQh + in), sdn = scalar_load(sdOh + in);
    if (t >= 2) {
      const BwdStageB1<D>& st = L.stB[(t - 2) % 3];
      const BwdExchange& X = L.xch[t & 1];
      const float w_dv = L.scl[t & 1][0] * sd0;
      const float w_dk = L.scl[t & 1][1] * sq0 * args.sm_scale;
      if constexpr (QSMOOTH) {
#pragma unroll
        for (int tt = 0; tt < NPB; tt++) dkacc[tt] = add_dk_bias(dkacc[tt], muq, cs[tt]);
      }
#pragma unroll
      for (int tt = 0; tt < NPB; tt++) {
        const int kbo = blk0 + tt;
        v16i av, ak;
#pragma unroll
        for (int r = 0; r < 16; r++) {
          av[r] = 0;
          ak[r] = 0;
        }
#pragma unroll
        for (int qs = 0; qs < 2; qs++) {
          const v4i a1 = *(const v4i*)(st.dot + ((qs * KS + cb) * 64 + lane) * 16);
          const v4i b1 = *(const v4i*)(X.pb + ((qs * 2 + kbo) * 64 + lane) * 16);
          av = __builtin_amdgcn_mfma_i32_32x32x32_i8(a1, b1, av, 0, 0, 0);
          const v4i a2 = *(const v4i*)(st.qt + ((qs * KS + cb) * 64 + lane) * 16);
          const v4i b2 = *(const v4i*)(X.dsb + ((qs * 2 + kbo) * 64 + lane) * 16);
          ak = __builtin_amdgcn_mfma_i32_32x32x32_i8(a2, b2, ak, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 16; r++) {
          dvacc[tt][r] = __builtin_fmaf((float)av[r], w_dv, dvacc[tt][r]);
          dkacc[tt][r] = __builtin_fmaf((float)ak[r], w_dk, dkacc[tt][r]);
        }
      }
    }
    sq0 = sq1;
    sd0 = sd1;
    sq1 = sqn;
    sd1 = sdn;
    __builtin_amdgcn_s_waitcnt(vmcnt_only(COPIES));          // the copies of the interval before have landed
    barrier_lds_only();
  }
  // ---- write dV, dK (bf16) ----
#pragma unroll
  for (int t = 0; t < NPB; t++) {
    const int key = 64 * j + 32 * (blk0 + t) + ll;
    unsigned short* pv = args.dV + chead + (size_t)key * rs + 32 * cb + 4 * h;
    unsigned short* pk = args.dK + chead + (size_t)key * rs + 32 * cb + 4 * h;
#pragma unroll
    for (int aa = 0; aa < 4; aa++) {
      v4us ov, ok;
#pragma unroll
      for (int b = 0; b < 4; b++) {
        ov[b] = float_to_bf16_bits(dvacc[t][4 * aa + b]);
        ok[b] = float_to_bf16_bits(dkacc[t][4 * aa + b]);
      }
      if (key < args.nvalid) {
        *(v4us*)(pv + 8 * aa) = ov;
        *(v4us*)(pk + 8 * aa) = ok;
      }
    }
  }
  __builtin_amdgcn_s_waitcnt(vmcnt_only(0));                 // (the copies past the last tile land before the LDS is given up)
}

// ---- four KV blocks per workgroup ----------------------------------------------------------------------
// sage_bwd_wide_kernel (d = 128).  The kernel above divides every tile between four waves twice over: a quadrant of S and dP
// each, then a channel block of dV and dK each, with psi(P) and psi(dS) handed over through LDS in between.  Here a wave owns 32
// KEYS: it forms S and dP of all 64 queries of a tile against them, and the quantised P and dS, one key per lane, are the B
// operands of its own dV and dK as they stand.  Two waves share a KV block and exchange the two tile maxima, nothing else; eight
// waves hold four KV blocks and share every staged Q block.  Against sage_bwd_kernel, per 64 x 64 tile: 100 instead of 128 KB of
// operands read from LDS and none written to it, half the staging copies, half the barriers, and 298 instead of 336 vector instructions per
// 32 x 32 piece.  The values, their order and so the bits are the same.
//
// Of a wave's 256 registers 128 hold dV and dK of its keys, 12 hold K^ (its last fragment lies in LDS: with 16 the allocator put
// one into scratch, whose reload waits for the copies in flight), and 64 carry P and dS from one interval to the next (psi needs
// the maxima of the whole tile).  The interval's products are laid out by hand, one between two scheduling barriers with the
// vector work that runs beside it, LDS operands two or three products ahead:
//   psi of the last tile  |  16 products of its dV, dK; beside them the INT32 -> FP32 updates of the product before, and
//   between those of dK the 8 products of S of this tile  |  16 products of dP; beside them P of this tile  |  dS, maxima
// The masked form of an interval (the first one, the diagonal, a partial KV block, the last one) has the same shape: it forms
// everything and masks what does not exist, because branches around its phases cost the allocator its registers as well (K^ in
// scratch: slower than the kernel above).
//
// Measured (us, two KV blocks per workgroup -> four): 64 heads of N = 2048 with the mask 206 -> 157, 32 of 4096 358 -> 273, 64 of
// 8192 2657 -> 2030; 8 heads of 8192 without 632 -> 468.  Steps on the way, the last of these shapes: K^ out of scratch 566 -> 498;
// dO copied as whole rows 488 -> 485; the copies dealt to the products instead of issued at the head of the interval, row statistics and
// exp2 one product ahead 485 -> 465; the younger wave of a SIMD first in phase B 462 -> 452.
// What bounds it: of about 7000 cycles an interval the vector instructions of a SIMD's two waves (1192, at 2.4 to 8.4 each) take
// 4300 and the 80 products 2560 of the matrix pipe; the rest is chains (psi, the end of dS) that two waves do not cover.
template <int D>
struct BwdStageA4 {           // operands of phase A for one Q block
  int8_t qf[64 * D];          // Q^  F fragments
  int8_t dof[128 * D];        // bf16 dO, row by row; 16-byte piece c of row r in slot c ^ (r & 15) of the row
  float nl2[64];              // -L * log2(e)
  float dl[64];               // -delta
};

template <int D, bool CAUSAL, bool QSMOOTH, int MODE = kBwdFused, bool KV128 = false>
__global__ void __launch_bounds__(512, 1) sage_bwd_wide_kernel(BwdArgs args) {
  static_assert(D == 128 && MODE != kBwdMaxOnly, "");
  constexpr int KS = D / 32;       // INT8 k-steps over d; channel blocks
  constexpr int KB = D / 16;       // bf16 k-steps over d
  constexpr int TILE = 64 * D;     // bytes of one INT8 tile
  constexpr int NF = TILE / 1024;  // 1 KiB fragments per INT8 tile
  constexpr int PPR = D / 8, RPF = 64 / PPR;   // 16-byte pieces of a bf16 row, rows per 1 KiB
  static_assert(NF == 8 && PPR == 16, "copies: one fragment of each kind per wave");
  struct Lds {
    BwdStageA4<D> stA[2];
    int8_t stB[2][2][TILE];        // [buffer][Q^, dO^]: TF fragments
    int8_t kst[8][1024];           // [wave]: the last of the KS fragments of K^ of its 32 keys (the others stay in registers)
    int8_t vst[8][32 * D * 2];     // [wave]: bf16 V of the wave's 32 keys as B fragments; at the end its dV, dK rows
    unsigned red[2][8][2];         // [tile parity][wave][max P, max |dS|] as bit patterns
    float bias[QSMOOTH ? 2 : 1][QSMOOTH ? 4 : 1][QSMOOTH ? 64 : 1];   // [buffer][KV block][key]: logit bias of a Q block
    float muq[QSMOOTH ? 2 : 1][QSMOOTH ? D : 1];                      // [buffer]: its mean
  };
  __shared__ __attribute__((aligned(256))) Lds L;

  const int N = args.N;
  const int nblk = N / kBlock;          // KV blocks
  const int nqblk = args.Nq / kBlock;   // Q blocks
  const int sb = CAUSAL ? args.shift_blocks : 0;
  const WorkItem wi = work_item(blockIdx.x, (nblk + 3) / 4, args.head_set);
  const int hl = wi.head;               // head within this launch
  const int bh = args.bh0 + hl;
  const int j0 = 4 * wi.item;           // small = most Q blocks under the causal mask: scheduled first

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ll = lane & 31, h = lane >> 5;
  const int kb = wave & 1;                        // 32-key half of the KV block
  const int j = j0 + (wave >> 1);
  const bool valid = j < nblk;
  const int jc = valid ? j : nblk - 1;            // clamped: a wave without a block still loads in bounds
  const int kvalid = min(64, args.nvalid - 64 * jc);

  const size_t qhead = (size_t)bh * args.Nq * D;
  const size_t rs = args.cv.row_stride, rsq = args.cvq.row_stride;
  const size_t chead = args.cv.row(bh, 0), cqhead = args.cvq.row(bh, 0);
  const float sKj = scalar_load(args.sK + (size_t)bh * nblk + jc);
  const float* sQh = args.sQ + (size_t)bh * nqblk;
  const float* sdOh = args.sdO + (size_t)bh * nqblk;
  // the walk: tile t is Q block itop - t, t = 0 .. T - 1 (at least one: the diagonal)
  const SingleWalk walk(nqblk, CAUSAL ? max(j0 - sb, 0) : 0);
  const int itop = walk.itop, T = walk.T;
  const size_t rsq_loop = walk.loop_row_step() ? rsq : 0;

  unsigned lane16 = lane * 16;
  // dO: this lane's piece of a fragment of four rows, in bytes (the wave copies fragments `wave` and `wave + 8`: rows 4 wave + ..
  // of either half)
  unsigned dO_lane = (unsigned)((lane / PPR) * 2 * rsq_loop + ((lane ^ (RPF * wave + lane / PPR)) & (PPR - 1)) * 16);
  v4i kfr[KS - 1];
  {
    const int8_t* p = args.KF + (size_t)bh * N * D + ((size_t)(2 * jc + kb) * KS) * 1024 + lane16;
#pragma unroll
    for (int s = 0; s < KS - 1; s++) kfr[s] = *(const v4i*)(p + s * 1024);
    async_copy_16(p + (KS - 1) * 1024, L.kst[wave]);
    // (a key row that does not exist re-reads the last one that does: its P is masked to zero)
    const unsigned short* pv = args.V + chead + (size_t)min(64 * jc + 32 * kb + ll, args.nvalid - 1) * rs + 8 * h;
#pragma unroll
    for (int s = 0; s < KB; s++) async_copy_16(pv + 16 * s, L.vst[wave] + s * 1024);
  }
  // the operands of phase A of tile 0: Q block itop may be the partial last one, so each row of dO is clamped
  {
    BwdStageA4<D>& st = L.stA[0];
    async_copy_16(args.QF + qhead + (size_t)itop * TILE + wave * 1024 + lane16, st.qf + wave * 1024);
#pragma unroll
    for (int f = wave; f < 2 * NF; f += 8) {
      const int r = RPF * f + lane / PPR;
      async_copy_16(args.dO + cqhead + (size_t)dO_row_clamped(64 * itop + r, args.nq_valid) * rsq + 8 * ((lane ^ r) & (PPR - 1)),
                    st.dof + f * 1024);
    }
    async_copy_4(((wave & 1) ? args.delta : args.nL2) + (size_t)bh * args.Nq + 64 * itop + lane, (wave & 1) ? st.dl : st.nl2);
    if constexpr (QSMOOTH) {
      async_copy_4(args.bias + ((size_t)bh * nqblk + itop) * N + 64 * jc + lane, L.bias[0][wave >> 1]);
    }
  }

  v16f dvacc[KS], dkacc[KS];
  float p[2][16], ds[2][16];     // [q half] P and dS of the wave's 64 x 32 piece of a tile, between its two intervals
#pragma unroll
  for (int r = 0; r < 16; r++) {
#pragma unroll
    for (int t = 0; t < KS; t++) dvacc[t][r] = dkacc[t][r] = 0.f;
    p[0][r] = p[1][r] = ds[0][r] = ds[1][r] = 0.f;
  }
  // maxima as bit patterns (non-negative floats order like theirs), kept in scalar registers
  int own_p = 0, own_d = 0;                                               // the wave's own, of that piece
  float cs = 0.f;                                                         // Q-smoothing: sm_scale * column sum of dS (see add_dk_bias)
  int prev_p = 0, prev_d = 0;                                             // kBwdPairedRows: the last tile's
  float sq = scalar_load(sQh + itop), sd = scalar_load(sdOh + itop);      // s_Q, s_dO of tile t
  float sq1 = 0.f, sd1 = 0.f;                                             // ... of tile t - 1
  barrier_all_memory();

  // Interval t: psi, dV, dK of tile t - 1 (HAS_Q: not in interval 0); S, dP, P, dS of tile t and copies of phase A's operands of tile
  // t + 1 (past the last tile that one again, never used) and of phase B's of tile t (HAS_A: not in interval T).  One barrier at its end.
  auto interval = [&](const int t, auto mask_tag, auto q_tag, auto a_tag) __attribute__((always_inline)) {
    constexpr bool MASK = decltype(mask_tag)::value;
    constexpr bool HAS_Q = decltype(q_tag)::value, HAS_A = decltype(a_tag)::value;
    const int iq = itop - (t - 1), ia = itop - t;
    // (the wave's tiles are the first ones of the walk; the comparisons with t hold wherever they are made: without them the compiler makes
    // two loops of it, for waves with a block and without, and has no registers for them)
    const bool act_q = HAS_Q && (!MASK || (t >= 1 && valid && (!CAUSAL || iq + sb >= j)));
    const bool act_a = HAS_A && (!MASK || (t < T && valid && (!CAUSAL || ia + sb >= j)));
    // (opaque: their extension to 64 bits and what is derived from the lane are formed here and not kept in registers)
    asm volatile("" : "+v"(lane16), "+v"(dO_lane));
    const int ll = (lane16 >> 4) & 31, h = lane16 >> 9;
    const BwdStageA4<D>& st = L.stA[t & 1];
    const int8_t* stq = L.stB[(t - 1) & 1][0] + lane16;
    const int8_t* stdo = L.stB[(t - 1) & 1][1] + lane16;
    const int8_t* qfp = st.qf + lane16;
    const int8_t* vbp = L.vst[wave] + lane16;
    const unsigned dofp = (unsigned)(uintptr_t)(lptr_t)st.dof + ll * 2 * D + ((h ^ ll) & (PPR - 1)) * 16;
    const unsigned(&R)[8][2] = L.red[(t - 1) & 1];
    unsigned pu, du;                                    // the other waves' maxima of the numerics block
    if constexpr (KV128) {
      const int g = wave & 4;
      pu = max(max(R[g][0], R[g + 1][0]), max(R[g + 2][0], R[g + 3][0]));
      du = max(max(R[g][1], R[g + 1][1]), max(R[g + 2][1], R[g + 3][1]));
    } else {
      pu = R[wave ^ 1][0];
      du = R[wave ^ 1][1];
    }
    // copy `part` of this wave's six (eight)
    constexpr int PARTS = QSMOOTH ? 8 : 6;
    const int in = walk.at(t + 1), ic = walk.at(t);
    auto copy_part = [&](int part) __attribute__((always_inline)) {
      BwdStageA4<D>& sa = L.stA[(t + 1) & 1];
      int8_t(&sbuf)[2][TILE] = L.stB[t & 1];
      const size_t toff = qhead + (size_t)in * TILE + wave * 1024, coff = qhead + (size_t)ic * TILE + wave * 1024;
      if (part == 0) copy_16(uniform(args.QF + toff) + lane16, sa.qf + wave * 1024);
      if (part == 1 || part == 2) {
        const int f = wave + 8 * (part - 1);
        copy_16(uniform(args.dO + cqhead + (size_t)(64 * in) * rsq + (size_t)(RPF * f) * rsq_loop) + dO_lane, sa.dof + f * 1024);
      }
      if (part == 3)
        copy_4(uniform(((wave & 1) ? args.delta : args.nL2) + (size_t)bh * args.Nq + 64 * in) + (lane16 >> 2), (wave & 1) ? sa.dl : sa.nl2);
      if (part == 4) copy_16(uniform(args.QT + coff) + lane16, sbuf[0] + wave * 1024);
      if (part == 5) copy_16(uniform(args.dOT + coff) + lane16, sbuf[1] + wave * 1024);
      // (the same values from both waves of a block, from four of the eight)
      if (QSMOOTH && part == 6) copy_4(uniform(args.bias + ((size_t)bh * nqblk + in) * N + 64 * jc) + (lane16 >> 2), L.bias[(t + 1) & 1][wave >> 1]);
      if (QSMOOTH && part == 7)
        copy_4(uniform(args.muQ + ((size_t)bh * nqblk + ic) * D + 64 * (wave & 1)) + (lane16 >> 2), L.muq[t & 1] + 64 * (wave & 1));
    };
    const float sqn = scalar_load(sQh + in), sdn = scalar_load(sdOh + in);
    __builtin_amdgcn_sched_barrier(0);
    if (!MASK || act_a || act_q) {
      // ---------------- psi of tile t - 1 ----------------
      v4i pf[2], df[2];            // [q half]: B operands of dV, dK, one key per lane
      float w_dv = 0.f, w_dk = 0.f;
      if constexpr (HAS_Q) {
        pu = max(pu, (unsigned)own_p);
        du = max(du, (unsigned)own_d);
        if constexpr (MODE == kBwdPairedRows) {
          // the other Q block of the numerics block: below (iq odd: the stored maxima of tile (iq - 1, j), and of its neighbour
          // in the 128-key block, where those tiles exist) or above (iq even: the last interval's)
          const unsigned bp = pu, bd = du;
          if (iq & 1) {
            const int jm = KV128 ? (jc & ~1) : jc;
            const float* tm = args.tmax + 2 * (((size_t)hl * nqblk + iq - 1) * args.ds_pitch + jm);
            if (!CAUSAL || jm <= iq - 1 + sb) {
              pu = max(pu, __float_as_uint(scalar_load(tm)));
              du = max(du, __float_as_uint(scalar_load(tm + 1)));
            }
            if (KV128 && jm + 1 < nblk && (!CAUSAL || jm + 1 <= iq - 1 + sb)) {
              pu = max(pu, __float_as_uint(scalar_load(tm + 2)));
              du = max(du, __float_as_uint(scalar_load(tm + 3)));
            }
          } else if (iq + 1 < nqblk) {
            pu = max(pu, (unsigned)prev_p);
            du = max(du, (unsigned)prev_d);
          }
          prev_p = __builtin_amdgcn_readfirstlane((int)bp);
          prev_d = __builtin_amdgcn_readfirstlane((int)bd);
        }
        const float bpm = __uint_as_float(pu), bdm = __uint_as_float(du);
        // the per-tile scales of P and dS are internal (never stored bit-exactly): 127/a via rcp
        const float rP = bpm > 0.f ? 127.0f * __builtin_amdgcn_rcpf(bpm) : 0.f;
        const float rS = bdm > 0.f ? 127.0f * __builtin_amdgcn_rcpf(bdm) : 0.f;
        const float sP = bpm * (1.0f / 127.0f), sS = bdm * (1.0f / 127.0f);
#pragma unroll
        for (int qh = 0; qh < 2; qh++)
#pragma unroll
          for (int aa = 0; aa < 4; aa++) {
            unsigned up = 0;
#pragma unroll
            for (int b = 0; b < 4; b++) up = __builtin_amdgcn_cvt_pk_u8_f32(p[qh][4 * aa + b] * rP, b, up);
            pf[qh][aa] = (int)up;
          }
#pragma unroll
        for (int qh = 0; qh < 2; qh++)
#pragma unroll
          for (int aa = 0; aa < 4; aa++) {
            unsigned ub[4];
#pragma unroll
            for (int b = 0; b < 4; b++) ub[b] = __float_as_uint(__builtin_fmaf(ds[qh][4 * aa + b], rS, kRoundMagic));
            df[qh][aa] = (int)(__builtin_amdgcn_perm(ub[1], ub[0], 0x0c0c0400u) | __builtin_amdgcn_perm(ub[3], ub[2], 0x04000c0cu));
          }
        w_dv = sP * sd1;
        w_dk = sS * sq1 * args.sm_scale;
        // (act_q whenever act_a, so always; the branch decides a register either way: none is in scratch with it here and without it there)
        if (MODE == kBwdPairedRows || !MASK || act_q) {
          // fragments (q half, kb) of the tile, as sage_bwd_kernel stores them
          const size_t tile = ((size_t)hl * nqblk + iq) * args.ds_pitch + j;
          const gbytes_t dst = uniform(args.dSq + tile * 4096 + kb * 1024);
          store_pair<2048>(dst, lane16, df[0], df[1], args.stream_ds);
          args.sdS[tile] = sS;       // (the same value from every lane)
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      // ---------------- dV, dK of tile t - 1 (phase B), S of tile t ----------------
      // Products u = 0 .. KS - 1: dV of channel block u, u = KS .. 2 KS - 1: dK of block u - KS, two steps each; those of dK have two
      // products of S (q half s / KS, step s % KS) between them: psi(P) is dead by then.
      first_for_younger_waves<1>(wave);
      struct Slot {
        int u, k, s;               // step k of product u, or (k < 0) product s of S
      };
      constexpr int NM = HAS_Q && HAS_A ? 6 * KS : HAS_Q ? 4 * KS : 2 * KS;
      auto slot = [](int m) constexpr {
        if (!HAS_Q) return Slot{KS, -1, m};
        if (!HAS_A) return Slot{m / 2, m % 2, 0};
        if (m < 2 * KS) return Slot{m / 2, m % 2, 0};
        const int n = m - 2 * KS;
        return n % 2 == 0 ? Slot{KS + n / 4, (n / 2) % 2, 0} : Slot{KS + n / 4, -1, n / 2};
      };
      v16i res[2], sacc[2], zero;
      v4i op[4], klast;
#pragma unroll
      for (int r = 0; r < 16; r++) zero[r] = 0;
      auto read_op = [&](int m) __attribute__((always_inline)) {
        const Slot sl = slot(m);
        op[m % 4] = sl.k >= 0 ? *(const v4i*)((sl.u < KS ? stdo : stq) + (sl.k * KS + sl.u % KS) * 1024) : *(const v4i*)(qfp + sl.s * 1024);
      };
      auto update = [&](int u, int r0, int r1) __attribute__((always_inline)) {
#pragma unroll
        for (int r = r0; r < r1; r++) {
          if (u >= KS) dkacc[u % KS][r] = __builtin_fmaf((float)res[u & 1][r], w_dk, dkacc[u % KS][r]);
          else dvacc[u][r] = __builtin_fmaf((float)res[u & 1][r], w_dv, dvacc[u][r]);
        }
      };
#pragma unroll
      for (int m = 0; m < 3; m++) read_op(m);
#pragma unroll
      for (int m = 0; m < NM; m++) {
        const Slot sl = slot(m);
        if (m + 3 < NM) read_op(m + 3);
        if (sl.k < 0 && sl.s % KS == KS - 2) klast = *(const v4i*)(L.kst[wave] + lane16);
        if (sl.k >= 0)
          res[sl.u & 1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(op[m % 4], sl.u < KS ? pf[sl.k] : df[sl.k], sl.k == 0 ? zero : res[sl.u & 1], 0, 0, 0);
        else
          sacc[sl.s / KS] = __builtin_amdgcn_mfma_i32_32x32x32_i8(op[m % 4], sl.s % KS == KS - 1 ? klast : kfr[sl.s % KS], sl.s % KS == 0 ? zero : sacc[sl.s / KS], 0, 0, 0);
        if (!HAS_Q && m < PARTS) copy_part(m);
        if (QSMOOTH && HAS_Q && m % 2 == 0 && m < 2 * KS)
          dkacc[m / 2] = add_dk_bias(dkacc[m / 2], L.muq[(t - 1) & 1][16 * m + ll], cs);
        if (HAS_Q && sl.u > 0 && (sl.u < KS || !HAS_A)) update(sl.u - 1, 8 * (m % 2), 8 * (m % 2) + 8);
        if (HAS_Q && HAS_A && sl.u >= KS) update(sl.u - 1, 4 * (m % 4), 4 * (m % 4) + 4);
        if (HAS_Q && HAS_A && m % 3 == 1 && m / 3 < PARTS) copy_part(m / 3);     // (dealt out: the waves do not queue up at the memory pipeline)
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (!HAS_A) {
        update(2 * KS - 1, 0, 16);
        first_for_younger_waves<0>(wave);
      } else {
        // ---------------- dP, P, dS of tile t ----------------
        const float c = sq * sKj * args.scale_log2e;
        v16f dp[2];
        v8bf da[3], vb[2];
        auto read_dO = [&](int m) __attribute__((always_inline)) {     // product m: q half m % 2, step m / 2
          da[m % 3] = *(const __attribute__((address_space(3))) v8bf*)(uintptr_t)((dofp ^ ((m / 2) * 32)) + (m & 1) * 64 * D);
        };
        auto read_V = [&](int s) __attribute__((always_inline)) { vb[s % 2] = *(const v8bf*)(vbp + s * 1024); };
        // -L log2e, LE elements at a time (with Q-smoothing there is no register for four)
        constexpr int LE = QSMOOTH ? 2 : 4;
        typedef float vle __attribute__((ext_vector_type(LE)));
        vle lst[2];
        auto read_L = [&](int g) __attribute__((always_inline)) {
          const int e = g * LE;
          lst[g & 1] = *(const vle*)(st.nl2 + 4 * h + 32 * (e >> 4) + 8 * ((e >> 2) & 3) + (e & 3));
        };
        float pm = 0.f, dm = 0.f;
        // masked: the rows of the tile below klow + 4 h (under the diagonal), or all 64 of a key or of a tile that does not exist
        // (in scalars first: as a choice of three it became branches around the products)
        const int kv = act_a ? kvalid : 0, off = CAUSAL && ia + sb == j ? 32 * kb : -128;
        const int klow = 32 * kb + ll >= kv ? 64 : ll - 4 * h + off;
        // P of element e (q half e / 16, register e % 16 = query 8 (r / 4) + 4 h + r % 4 of it), in three steps that run one product apart
        const float bias_l = QSMOOTH ? L.bias[t & 1][wave >> 1][32 * kb + ll] : 0.f;
        auto form_x = [&](int e) __attribute__((always_inline)) {
          const float l = lst[(e / LE) & 1][e % LE];
          p[e >> 4][e & 15] = __builtin_fmaf((float)sacc[e >> 4][e & 15], c, QSMOOTH ? bias_l + l : l);
        };
        auto form_p = [&](int e) __attribute__((always_inline)) {
          const int qh = e >> 4, r = e & 15;
          const float pv = __builtin_amdgcn_exp2f(p[qh][r]);
          p[qh][r] = MASK && 32 * qh + 2 * (r & ~3) + (r & 3) < klow ? 0.f : pv;
        };
        auto form_max = [&](int e) __attribute__((always_inline)) { pm = fmaxf(fmaxf(p[e >> 4][e & 15], p[e >> 4][(e & 15) + 1]), pm); };
        read_V(0);
        read_dO(0);
        read_dO(1);
        read_L(0);
        // dS = P o (dP - delta): the chains start from -delta of the rows a lane's registers hold
        auto read_delta = [&](int qh) __attribute__((always_inline)) {
#pragma unroll
          for (int aa = 0; aa < 4; aa++) {
            const v4f d4 = *(const v4f*)(st.dl + 32 * qh + 4 * h + 8 * aa);
#pragma unroll
            for (int b = 0; b < 4; b++) dp[qh][4 * aa + b] = d4[b];
          }
        };
        read_delta(0);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (HAS_Q) update(2 * KS - 1, 0, 16);         // (while those reads are under way; its operands' registers go to the second chain)
        __builtin_amdgcn_sched_barrier(0);
        read_delta(1);
#pragma unroll
        for (int m = 0; m < 2 * KB; m++) {
          if (m + 2 < 2 * KB) read_dO(m + 2);
          if (m % 2 == 0 && m / 2 + 1 < KB) read_V(m / 2 + 1);
          if (2 * m % LE == 0 && 2 * m + LE < 32) read_L(2 * m / LE + 1);
          dp[m & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(da[m % 3], vb[(m / 2) % 2], dp[m & 1], 0, 0, 0);
          // (first through most of dP too: its operands are read under the older wave's dK.  Dropped at product 0, 3, 7, 11, 16: 64
          // heads of N = 8192 with the mask 1997, 1991, 1986, 1965, 2000 us)
          if (m == 11) first_for_younger_waves<0>(wave);
          if (m >= 2) form_max(2 * m - 4);
          if (m >= 1) {
            form_p(2 * m - 2);
            form_p(2 * m - 1);
          }
          form_x(2 * m);
          form_x(2 * m + 1);
          __builtin_amdgcn_sched_barrier(0);
        }
        form_max(28);
        form_p(30);
        form_p(31);
        form_max(30);
#pragma unroll
        for (int qh = 0; qh < 2; qh++)
#pragma unroll
          for (int r = 0; r < 16; r += 2) {
#pragma unroll
            for (int b = r; b < r + 2; b++) {
              ds[qh][b] = p[qh][b] * dp[qh][b];
              if constexpr (MASK) ds[qh][b] = act_a ? ds[qh][b] : 0.f;   // (no tile: nothing, whatever the stage holds)
            }
            dm = fmaxf(fmaxf(fabsf(ds[qh][r]), fabsf(ds[qh][r + 1])), dm);
          }
        if constexpr (QSMOOTH) {
          float cs0 = 0.f, cs1 = 0.f;
#pragma unroll
          for (int r = 0; r < 16; r++) {
            cs0 += ds[0][r];
            cs1 += ds[1][r];
          }
          cs = (cs0 + cs1) * args.sm_scale;
        }
        own_p = __builtin_amdgcn_readfirstlane(__float_as_int(wave_max_nonneg_f32(pm)));
        own_d = __builtin_amdgcn_readfirstlane(__float_as_int(wave_max_nonneg_f32(dm)));
        L.red[t & 1][wave][0] = (unsigned)own_p;     // (the same pair from every lane)
        L.red[t & 1][wave][1] = (unsigned)own_d;
      }
    } else if constexpr (HAS_A) {
#pragma unroll
      for (int part = 0; part < PARTS; part++) copy_part(part);
      if constexpr (KV128) L.red[t & 1][wave][0] = L.red[t & 1][wave][1] = 0u;   // nothing for the neighbour's block maxima
    }
    sq1 = sq;
    sd1 = sd;
    sq = sqn;
    sd = sdn;
    if constexpr (HAS_A) barrier_all_memory();   // the interval's LDS traffic, copies and stores are complete
  };
  // unmasked intervals: both tiles exist in full, tile t above the diagonal
  const int t_steady_end = !valid || kvalid < 64 ? 0 : CAUSAL ? min(itop + sb - j, T - 1) : T - 1;
  // the first interval, the unmasked ones, the others (written so that their masked form is there once), the last one.  The first and
  // the last are half an interval each: in the masked form, as they were, each wasted the other half (64 heads of N = 2048 with the
  // mask 136.3 -> 129.2 us, 32 of 4096 236 -> 228.5, 64 of 8192 1970 -> 1900, 8 of 8192 without 438 -> 429, the dP priority included).
  interval(0, std::true_type{}, std::false_type{}, std::true_type{});
#pragma clang loop unroll(disable)
  for (int t = 1; t < T;) {
#pragma clang loop unroll(disable)
    for (; t < t_steady_end; t++) interval(t, std::false_type{}, std::true_type{}, std::true_type{});
    if (t < T) interval(t++, std::true_type{}, std::true_type{}, std::true_type{});
  }
  interval(T, std::true_type{}, std::true_type{}, std::false_type{});

  if (!valid) return;
  // ---- write dV, then dK (bf16): through the wave's own V stage (nobody else reads it), so that whole rows leave.  Piece c of row
  // r lies in slot c ^ (r & 15) of its row. ----
  int8_t* stg = L.vst[wave];
  const int key0 = 64 * j + 32 * kb;
#pragma unroll
  for (int which = 0; which < 2; which++) {
    const v16f(&acc)[KS] = which == 0 ? dvacc : dkacc;
    unsigned short* out = (which == 0 ? args.dV : args.dK) + chead;
#pragma unroll
    for (int cb = 0; cb < KS; cb++)
#pragma unroll
      for (int aa = 0; aa < 4; aa++) {
        v4us o;
#pragma unroll
        for (int b = 0; b < 4; b++) o[b] = float_to_bf16_bits(acc[cb][4 * aa + b]);
        *(v4us*)(stg + ll * 2 * D + (((4 * cb + aa) ^ ll) & (PPR - 1)) * 16 + 8 * h) = o;
      }
    // (one wave: its LDS operations complete in order)
#pragma unroll
    for (int k = 0; k < 32 / RPF; k++) {
      const int r = RPF * k + lane / PPR;
      const v8us piece = *(const v8us*)(stg + r * 2 * D + ((lane ^ r) & (PPR - 1)) * 16);
      if (key0 + r < args.nvalid) stream_store((v8us*)(out + (size_t)(key0 + r) * rs + 8 * (lane % PPR)), piece);
    }
  }
}

// ---------------------------------------------------------------------------------
// dQ_i = sum_j (dS^_ij K^_j) * s_dS(i,j) * s_K(j) * sm_scale        (Algorithm 2, the dQ line)
// A = the stored psi(dS) fragments, transposed here, B = K^ in TF layout.
struct DqArgs {
  const int8_t* dSq;
  int ds_pitch;         // tiles per Q-block row of dSq
  const float* sdS;
  const int8_t* KT;
  const float* sK;
  unsigned short* dQ;   // bf16, rows addressed through `cv` (dense [BH, N_q, D] or the caller's token-major tensor)
  RowView cv;
  int BH, N, bh0;       // N = rows of the K-like workspace tensors (a multiple of 64)
  int Nq;               // rows of the Q-like ones
  int nvalid;           // query rows >= nvalid do not exist
  int shift_blocks;     // causal: Q block i sees KV blocks j <= i + shift_blocks
  int head_set;         // heads per XCD whose work items are interleaved (see work_item)
  int last_first;       // the last heads first: their tiles are still cached (see ds_traffic)
  float sm_scale;       // times 2^13
};

// The INT32 sums arrive as a 2^-26 (mfma_from_bias).  Half of that is made up in the weights (sm_scale), half at the end: with all of it at
// the end the sums of gradients below 2^-100 were denormal.  (A weight is then 2^13 times what a converted sum's would be: where
// s_dS s_K scale is 2^115 and more it is infinite, though the gradient of small codes might not be.)
constexpr float kDqWeight = 8192.0f;
static_assert(kDqWeight * kDqWeight == kTwo26, "the two halves");

// A workgroup of 4 waves owns TWO Q blocks (128 queries) and walks the KV blocks j; wave (Q block, row half)
// owns 32 query rows and ALL d channels.  A stored psi(dS) fragment holds one KEY per lane and 16 queries in
// its bytes (the form the backward kernel's own products need); the product over keys needs one QUERY per
// lane, so each fragment is transposed on arrival by one MFMA against a permutation matrix: read as an A
// operand it is the matrix (key, permuted query), and the accumulator comes back with lane = query and
// registers = keys in the order of the TF layout of K^; the low bytes of the INT32 results are the codes.
// Each wave streams its own 2 KiB per tile from HBM straight into registers (one 16-byte load per lane
// and fragment, nothing shared, no LDS): kStages tiles ahead.  The K^ tile (TF layout, from L2) is
// shared by the four waves and travels global -> LDS asynchronously through a ring that runs the same
// number of stages ahead, together with the three scales of the stage; one barrier per stage.  Both
// streams are issued by every wave in the same order and complete in order, so one count of outstanding
// memory operations (`s_waitcnt vmcnt`) covers the K^ copies and the compiler's own waits cover the
// registers.  Three workgroups share a CU: about 96 KiB of psi(dS) in flight per CU.
// (Every lane takes part in the scale copy: a memory operation under a lane mask sits behind a branch,
// and with a path that skips it the compiler stops counting the loads in flight and waits for all of
// them before each use.)  Measured, 64 heads of N = 8192 with the mask: with cached loads, conversions and cached stores the
// kernel took 0.54 ms, its psi(dS) stream alone (no arithmetic, no K^ copies) 0.51, where a plain read stream over the same
// bytes reaches 5.6 TB/s on this GPU; ring depths 3 to 7 and two or three workgroups per CU changed nothing.  What did: psi(dS)
// stored and loaded past the caches (see ds_traffic), 538 -> 520 us, dQ, dK and dV stored past them (what a kernel leaves dirty in
// the L2 is written back at its end) -> 506, and a subtraction in place of the conversion -> 491.
// STREAM: psi(dS) is loaded past the caches.
template <int D, bool CAUSAL, bool STREAM>
__global__ void __launch_bounds__(256, 3) sage_bwd_dq_kernel(DqArgs args) {
  constexpr int KS = D / 32;               // channel blocks
  constexpr int TILE = 64 * D;             // bytes of one K^ tile
  constexpr int DSB = 4096;                // bytes of one psi(dS) tile
  constexpr int kStages = 4;               // stages in flight (3 to 7 measured the same)
  constexpr int NS = kStages + 1;          // ring slots
  constexpr int KSLOT = TILE + 256;        // K^ tile | s_dS of Q block 0, of Q block 1, s_K (lanes 3.. repeat s_K)
  constexpr int KC = TILE / 4096;          // K^ copies per wave and stage (the tile's 1 KiB fragments dealt to 4 waves)
  constexpr int OPS = 2 + KC + 1;          // memory operations per wave and stage: 2 psi(dS) loads, K^ copies, scales

  __shared__ __attribute__((aligned(16))) int8_t lds[NS * KSLOT];

  const int g = blockIdx.x;
  const int N = args.N;
  const int nblk = N / kBlock;                         // KV blocks
  const int nqblk = args.Nq / kBlock;                  // Q blocks
  const int sb = CAUSAL ? args.shift_blocks : 0;
  const int npair = (nqblk + 1) / 2;
  const WorkItem wi = work_item(g, npair, args.head_set);
  const int hl = args.last_first ? args.BH - 1 - wi.head : wi.head;
  const int bh = args.bh0 + hl;
  const int i0 = 2 * (npair - 1 - wi.item);            // longest rows first under the causal mask
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ll = lane & 31, h = lane >> 5;
  const int iq = wave >> 1, qb = wave & 1;             // Q block of the pair, 32-row half of it
  const bool valid = i0 + iq < nqblk;
  const int i = valid ? i0 + iq : i0;                  // clamped: the loads stay in bounds
  const int i1 = i0 + 1 < nqblk ? i0 + 1 : i0;
  const size_t head = (size_t)bh * N * D;
  const int n_j = CAUSAL ? min(i0 + 2 + sb, nblk) : nblk;            // stages of the workgroup
  const int j_last = CAUSAL ? i + sb : nblk - 1;       // last tile of this wave's Q block that was written

  // this wave's fragments of tile (i, j): (row half qb, key step 0 / 1) at j * DSB, + 1024
  const int8_t* dsw = args.dSq + ((size_t)hl * nqblk + i) * args.ds_pitch * DSB + qb * 2048 + lane * 16;
  const int8_t* kth = args.KT + head + wave * 1024 + lane * 16;
  // per stage lanes 0, 1, 2 fetch s_dS of Q block 0, s_dS of Q block 1, s_K
  const size_t sc_off = lane == 0 ? ((size_t)hl * nqblk + i0) * args.ds_pitch : ((size_t)hl * nqblk + i1) * args.ds_pitch;
  const float* sc_src = lane < 2 ? args.sdS + sc_off : args.sK + (size_t)bh * nblk;

  // Stage indices past the end are clamped: the loads then re-read the last stage (into registers or a
  // slot that nobody reads any more), and every wave issues the same operations in every iteration.
  auto load_ds = [&](int j, v4i (&a)[2]) __attribute__((always_inline)) {
    const int jc = j < j_last ? j : j_last;
    const int8_t* p = dsw + (size_t)jc * DSB;
    a[0] = STREAM ? stream_load((const v4i*)p) : *(const v4i*)p;
    a[1] = STREAM ? stream_load((const v4i*)(p + 1024)) : *(const v4i*)(p + 1024);
  };
  auto load_k = [&](int j, int sl) __attribute__((always_inline)) {
    const int jc = dq_stage(j, n_j);
    const int8_t* src = kth + (size_t)jc * TILE;
    int8_t* dst = lds + sl * KSLOT + wave * 1024;
    async_copy_16(src, dst);
    if constexpr (KC == 2) async_copy_16(src + 4096, dst + 4096);
    async_copy_4(sc_src + jc, lds + sl * KSLOT + TILE);   // (the same values from every wave; lanes 2.. all carry s_K)
  };

  v16f acc[KS];
#pragma unroll
  for (int cb = 0; cb < KS; cb++)
#pragma unroll
    for (int r = 0; r < 16; r++) acc[cb][r] = 0.f;

  // B operand of the transposing MFMA: a stored fragment, read as an A operand, has contraction index
  // k = 16 h + 4 a + b for the query 8 a + 4 h + b; column n of the permutation matrix picks the k that
  // stands for query n.  Lane (n, hh) holds k = 16 hh + t in byte t.
  v4i tperm;
#pragma unroll
  for (int aa = 0; aa < 4; aa++) {
    unsigned u = 0;
#pragma unroll
    for (int b = 0; b < 4; b++) u |= (unsigned)((8 * aa + 4 * h + b) == ll) << (8 * b);
    tperm[aa] = (int)u;
  }
  auto transposed = [&](const v4i& f) __attribute__((always_inline)) {
    v16i z;
#pragma unroll
    for (int r = 0; r < 16; r++) z[r] = 0;
    const v16i tr = __builtin_amdgcn_mfma_i32_32x32x32_i8(f, tperm, z, 0, 0, 0);
    v4i o;
#pragma unroll
    for (int aa = 0; aa < 4; aa++) {
      const unsigned lo = __builtin_amdgcn_perm((unsigned)tr[4 * aa + 1], (unsigned)tr[4 * aa], 0x0c0c0400u);
      const unsigned hi = __builtin_amdgcn_perm((unsigned)tr[4 * aa + 3], (unsigned)tr[4 * aa + 2], 0x04000c0cu);
      o[aa] = (int)(lo | hi);
    }
    return o;
  };

  v4i a[kStages][2];
#pragma unroll
  for (int s = 0; s < kStages; s++) {
    load_ds(s, a[s]);
    load_k(s, s);
    compiler_fence();                      // the waits below count operations in issue order
  }
  static_assert((kStages - 1) * OPS < 64, "vmcnt has six bits");
  __builtin_amdgcn_s_waitcnt(vmcnt_only((kStages - 1) * OPS));   // stage 0 has landed
  barrier_lds_only();

  // Iteration j: contract stage j (registers a[j % kStages], ring slot j % NS), then start stage
  // j + kStages into the same registers and into the slot that stage j - 1 occupied (every wave is past
  // the barrier that ended iteration j - 1); before the barrier at the end, wait until this wave's
  // copies of stage j + 1 have landed (everything but the kStages - 1 youngest stages).
  // The loop is unrolled over the kStages register sets and runs whole rounds (the stages past n_j only
  // keep the counts even: clamped loads, no arithmetic), so that every path through the body issues the
  // same memory operations and the compiler's count of the loads in flight stays exact.
  int sk = 0;                              // slot of stage j
  for (int j0 = 0; j0 < n_j; j0 += kStages) {
#pragma unroll
    for (int s = 0; s < kStages; s++) {
      const int j = j0 + s;
      if (j < n_j && valid && (!CAUSAL || j <= i + sb)) {
        const int8_t* kp = lds + sk * KSLOT;
        const float* sc = (const float*)(kp + TILE);
        const float w = sc[iq] * sc[2] * args.sm_scale;
        const v4i a0 = transposed(a[s][0]), a1 = transposed(a[s][1]);
#pragma unroll
        for (int cb = 0; cb < KS; cb++) {
          const v4i b0 = *(const v4i*)(kp + cb * 1024 + lane * 16);
          const v4i b1 = *(const v4i*)(kp + (KS + cb) * 1024 + lane * 16);
          // (the sum less the bias is a 2^-26 exactly, and a subtraction takes half the time of a conversion)
          v16i q = mfma_from_bias(a0, b0);
          q = __builtin_amdgcn_mfma_i32_32x32x32_i8(a1, b1, q, 0, 0, 0);
#pragma unroll
          for (int r = 0; r < 16; r++) acc[cb][r] = __builtin_fmaf(__int_as_float(q[r]) - kBiasC0, w, acc[cb][r]);
        }
      }
      load_ds(j + kStages, a[s]);
      load_k(j + kStages, sk == 0 ? NS - 1 : sk - 1);
      __builtin_amdgcn_s_waitcnt(vmcnt_only((kStages - 1) * OPS));
      barrier_lds_only();
      sk = sk == NS - 1 ? 0 : sk + 1;
    }
  }
  barrier_all_memory();    // the clamped copies past the last stage have landed before the ring is reused
  // ---- write dQ (bf16): the accumulators hold one channel per lane and 16 query rows in registers, so
  // the two 64 x D blocks go through LDS (the ring is drained) and leave as 16-byte row pieces ----
  constexpr int LDQ = D + 8;                                   // padded row, in bf16 elements
  static_assert(2 * 64 * LDQ * 2 <= NS * KSLOT, "the dQ staging must fit the ring");
  unsigned short* stg = (unsigned short*)lds;                  // [Q block][row][LDQ]
  if (valid) {
#pragma unroll
    for (int cb = 0; cb < KS; cb++)
#pragma unroll
      for (int aa = 0; aa < 4; aa++)
#pragma unroll
        for (int b = 0; b < 4; b++)
          stg[(iq * 64 + 32 * qb + 8 * aa + 4 * h + b) * LDQ + 32 * cb + ll] = float_to_bf16_bits(acc[cb][4 * aa + b] * kDqWeight);
  }
  barrier_lds_only();
  constexpr int CPR = D / 8;                                   // 16-byte pieces per row
  for (int c = tid; c < 2 * 64 * CPR; c += 256) {
    const int qblk = c / (64 * CPR), row = (c / CPR) % 64, pc = c % CPR;
    if (i0 + qblk < nqblk && 64 * (i0 + qblk) + row < args.nvalid)
      stream_store((v8us*)(args.dQ + args.cv.row(bh, 64 * (i0 + qblk) + row) + 8 * pc), *(const v8us*)(stg + (qblk * 64 + row) * LDQ + 8 * pc));
  }
}

// dQ of calls whose launch of the kernel above does not fill the machine: it then takes as long as its longest chain of stages, at
// about 0.7 us a stage, most of it the latency of one wave's transposition, products and updates in turn.  Here a workgroup owns ONE
// Q block and takes two stages (KV blocks) an interval; wave (row half, channel block of 32) owns 32 x 32 of dQ, eight waves at d =
// 128 and four at d = 64, and a fragment of psi(dS) is transposed by one wave only, an interval ahead, and handed on through LDS:
// 0.4 us a stage.  (An interval first issues all its LDS reads and the transposing product, and the loads behind them; with the
// transposition hoisted over the barrier of the interval before by the compiler, which then waited for every load in flight, a stage
// took 0.5.)  Twice the copies of K^ of the kernel above are what a full machine pays.  The order of the sums is that of the kernel
// above: the same bits. us, kernel above -> this one, with the mask: 8 heads of N = 4096 48.5 -> 25.5, 24 of 2048 28.6 -> 21.5, 6 of
// 9000 104 -> 69, 2 of 1368 21.0 -> 12.0, 6 of 4467, d = 64, 35.0 -> 24.1; without: 6 of 2297 29.8 -> 16.5, 12 of 768 14.5 -> 9.3
// (the rule: use_dq_split).
template <int D, bool CAUSAL, bool STREAM>
__global__ void __launch_bounds__(4 * D, D == 128 ? 4 : 2) sage_bwd_dq_split_kernel(DqArgs args) {
  constexpr int KS = D / 32;               // channel blocks
  constexpr int NW = 2 * KS;               // waves
  constexpr int FW = 8 / NW;               // psi(dS) fragments of an interval that a wave transposes
  constexpr int TILE = 64 * D;             // bytes of one K^ tile
  constexpr int DSB = 4096;                // bytes of one psi(dS) tile
  constexpr int NS = 3;                    // ring slots, of two stages each: two intervals run ahead
  constexpr int KSLOT = 2 * TILE;          // two K^ tiles
  constexpr int OPS = FW + 2;              // memory operations per wave and interval: psi(dS), K^ copies

  struct Lds {
    __attribute__((aligned(16))) int8_t ring[NS * KSLOT];
    __attribute__((aligned(16))) int8_t frag[2][2 * DSB];     // [interval parity]: the transposed tiles
  };
  __shared__ __attribute__((aligned(16))) Lds L;

  const int N = args.N;
  const int nblk = N / kBlock;                         // KV blocks
  const int nqblk = args.Nq / kBlock;                  // Q blocks
  const WorkItem wi = work_item(blockIdx.x, nqblk, args.head_set);
  const int hl = args.last_first ? args.BH - 1 - wi.head : wi.head;
  const int bh = args.bh0 + hl;
  const int i = nqblk - 1 - wi.item;                   // longest rows first under the causal mask
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ll = lane & 31, h = lane >> 5;
  const int qb = wave / KS, cb = wave % KS;            // row half, channel block
  const int n_j = CAUSAL ? min(i + args.shift_blocks + 1, nblk) : nblk;         // stages

  const size_t row = ((size_t)hl * nqblk + i) * args.ds_pitch;
  const int8_t* dsw = args.dSq + row * DSB + (wave & 3) * 1024;
  const int8_t* kth = args.KT + (size_t)bh * N * D + wave * 1024;
  const float *sds = args.sdS + row, *sks = args.sK + (size_t)bh * nblk;
  const unsigned lane16 = lane * 16;

  // Stages past the end are clamped (see sage_bwd_dq_kernel).
  auto stage = [&](int j) { return dq_stage(j, n_j); };
  // fragment wave + NW f of the interval's eight: four a stage
  auto load_ds = [&](int m, v4i (&a)[FW]) __attribute__((always_inline)) {
#pragma unroll
    for (int f = 0; f < FW; f++) {
      const int j = stage(2 * m + (FW == 1 ? wave >> 2 : f));
      const __attribute__((address_space(1))) v4i* p = (const __attribute__((address_space(1))) v4i*)(uniform(dsw + (size_t)j * DSB) + lane16);
      a[f] = STREAM ? __builtin_nontemporal_load(p) : *p;
    }
  };
  auto load_k = [&](int m, int sl) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < 2; k++)
      copy_16(uniform(kth + (size_t)stage(2 * m + k) * TILE) + lane16, L.ring + sl * KSLOT + k * TILE + wave * 1024);
  };

  v16f acc;
#pragma unroll
  for (int r = 0; r < 16; r++) acc[r] = 0.f;

  // (the transposing product: see sage_bwd_dq_kernel)
  v4i tperm;
#pragma unroll
  for (int aa = 0; aa < 4; aa++) {
    unsigned u = 0;
#pragma unroll
    for (int b = 0; b < 4; b++) u |= (unsigned)((8 * aa + 4 * h + b) == ll) << (8 * b);
    tperm[aa] = (int)u;
  }
  auto transposed = [&](const v4i& f) __attribute__((always_inline)) {
    v16i z;
#pragma unroll
    for (int r = 0; r < 16; r++) z[r] = 0;
    return __builtin_amdgcn_mfma_i32_32x32x32_i8(f, tperm, z, 0, 0, 0);
  };
  auto hand_on = [&](const v16i (&tr)[FW], int parity) __attribute__((always_inline)) {
#pragma unroll
    for (int f = 0; f < FW; f++) {
      v4i o;
#pragma unroll
      for (int aa = 0; aa < 4; aa++) {
        const unsigned lo = __builtin_amdgcn_perm((unsigned)tr[f][4 * aa + 1], (unsigned)tr[f][4 * aa], 0x0c0c0400u);
        const unsigned hi = __builtin_amdgcn_perm((unsigned)tr[f][4 * aa + 3], (unsigned)tr[f][4 * aa + 2], 0x04000c0cu);
        o[aa] = (int)(lo | hi);
      }
      *(v4i*)(L.frag[parity] + (wave + NW * f) * 1024 + lane * 16) = o;
    }
  };
  // s_dS s_K of the two stages of an interval, through the scalar cache, an interval ahead
  v2f scale;
  auto load_scale = [&](int m) __attribute__((always_inline)) {
    const int j = stage(2 * m), j1 = stage(2 * m + 1);
    scale[0] = scalar_load(sds + j) * scalar_load(sks + j) * args.sm_scale;
    scale[1] = scalar_load(sds + j1) * scalar_load(sks + j1) * args.sm_scale;
  };
  // the operands of the interval's two products of each stage
  struct Operands {
    v4i a0[2], a1[2], b0[2], b1[2];
  };
  auto read = [&](int sl, int parity, Operands& x) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < 2; k++) {
      const int8_t* ap = L.frag[parity] + k * DSB + qb * 2048 + lane * 16;
      const int8_t* bp = L.ring + sl * KSLOT + k * TILE + cb * 1024 + lane * 16;
      x.a0[k] = *(const v4i*)ap;
      x.b0[k] = *(const v4i*)bp;
      x.a1[k] = *(const v4i*)(ap + 1024);
      x.b1[k] = *(const v4i*)(bp + KS * 1024);
    }
  };
  auto add = [&](const v16i& q, float w) __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < 16; r++) acc[r] = __builtin_fmaf(__int_as_float(q[r]) - kBiasC0, w, acc[r]);
  };

  v4i first[FW], a[2][FW];                 // a[m & 1]: the fragments of interval m
  load_scale(0);
  load_ds(0, first);
#pragma unroll
  for (int m = 0; m < 2; m++) {
    load_ds(m + 1, a[(m + 1) & 1]);
    load_k(m, m);
    compiler_fence();                      // the waits below count operations in issue order
  }
  v16i tr[FW];
#pragma unroll
  for (int f = 0; f < FW; f++) tr[f] = transposed(first[f]);
  hand_on(tr, 0);
  __builtin_amdgcn_s_waitcnt(vmcnt_only(OPS));   // interval 0 has landed
  barrier_lds_only();

  // Interval m: transpose the fragments of interval m + 1, contract stages 2m and 2m + 1, start the loads of m + 3 and the copies of m + 2
  // (into the slot of m - 1: every wave is past the barrier that ended it), wait for the copies of m + 1.
  int sl = 0, m = 0;                       // slot of interval m
  auto interval = [&](auto parity_tag) __attribute__((always_inline)) {
    constexpr int P = decltype(parity_tag)::value;
    Operands x;
    read(sl, P, x);
#pragma unroll
    for (int f = 0; f < FW; f++) tr[f] = transposed(a[P ^ 1][f]);
    __builtin_amdgcn_sched_barrier(0);
    v16i q[2];
    q[0] = mfma_from_bias(x.a0[0], x.b0[0]);
    q[0] = __builtin_amdgcn_mfma_i32_32x32x32_i8(x.a1[0], x.b1[0], q[0], 0, 0, 0);
    hand_on(tr, P ^ 1);
    load_ds(m + 3, a[P ^ 1]);
    __builtin_amdgcn_sched_barrier(0);
    q[1] = mfma_from_bias(x.a0[1], x.b0[1]);
    q[1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(x.a1[1], x.b1[1], q[1], 0, 0, 0);
    load_k(m + 2, sl == 0 ? NS - 1 : sl - 1);
    __builtin_amdgcn_sched_barrier(0);
    const v2f w = scale;
    load_scale(m + 1);
    add(q[0], w[0]);
    __builtin_amdgcn_sched_barrier(0);
    add(q[1], w[1]);
    __builtin_amdgcn_s_waitcnt(vmcnt_only(OPS));
    barrier_lds_only();
    __builtin_amdgcn_sched_barrier(0);
    sl = sl == NS - 1 ? 0 : sl + 1;
    m++;
  };
  const int pairs = n_j / 2;
  while (m + 1 < pairs) {
    interval(std::integral_constant<int, 0>{});
    interval(std::integral_constant<int, 1>{});
  }
  auto last = [&](int parity) __attribute__((always_inline)) {
    Operands x;
    read(sl, parity, x);
    v16i q = mfma_from_bias(x.a0[0], x.b0[0]);
    add(__builtin_amdgcn_mfma_i32_32x32x32_i8(x.a1[0], x.b1[0], q, 0, 0, 0), scale[0]);
  };
  if (m < pairs) {
    interval(std::integral_constant<int, 0>{});
    if (n_j & 1) last(1);
  } else if (n_j & 1) {
    last(0);
  }
  barrier_all_memory();    // the clamped copies past the last stage have landed before the ring is reused
  constexpr int LDQ = D + 8;                                   // padded row, in bf16 elements
  static_assert(64 * LDQ * 2 <= NS * KSLOT, "the dQ staging must fit the ring");
  unsigned short* stg = (unsigned short*)L.ring;               // [row][LDQ]
#pragma unroll
  for (int aa = 0; aa < 4; aa++)
#pragma unroll
    for (int b = 0; b < 4; b++) stg[(32 * qb + 8 * aa + 4 * h + b) * LDQ + 32 * cb + ll] = float_to_bf16_bits(acc[4 * aa + b] * kDqWeight);
  barrier_lds_only();
  constexpr int CPR = D / 8;                                   // 16-byte pieces per row
#pragma unroll
  for (int k = 0; k < 64 * CPR / (64 * NW); k++) {
    const int c = tid + 64 * NW * k, r = c / CPR, pc = c % CPR;
    if (64 * i + r < args.nvalid) stream_store((v8us*)(args.dQ + args.cv.row(bh, 64 * i + r) + 8 * pc), *(const v8us*)(stg + r * LDQ + 8 * pc));
  }
}

}  // namespace sage
