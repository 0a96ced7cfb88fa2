// Backward for short heads: the pre-pass, dV, dK and dQ in one launch.
//
// A workgroup of eight waves takes a whole head of at most NB blocks of 64 queries and NB of 64 keys.  It quantises dO (and Q and K
// where the forward has not left them: SHARE) and holds every code in LDS.  Four waves a KV block form a quarter of S, dP, P and dS of
// each of its tiles, psi(P) and psi(dS) of all tiles go through LDS (dS in two orders, one query per lane for dQ's product), and then
// each wave adds a block of channels of dQ, and of dV and dK, the Q blocks from the last down.  Values, their order and so
// the bits are those of the other forms; what those leave in the workspace for the inspection hooks is left here too.
//
// Such a backward took three launches, each of which is over in about the time that it takes to begin and to end.  Of 33000 cycles with
// two blocks at d = 128 the loads took 8000, dV and dK stored by 8 bytes a lane 4000, and the two Q blocks one after the other 11000: all
// tiles at once and gradients in whole rows 27.3 -> 24.8 us a step of 8 heads of N = 128, 131 -> 118 of 2048 of N = 64.
#pragma once

#include "common.h"
#include "bwd_kernel.h"
#include "fwd_short_kernel.h"

namespace sage {

// (products and sums are rounded apart, as in the other forms, but where an FMA is written)
#pragma clang fp contract(off)

struct ShortBwdArgs {
  const unsigned short *Q, *K, *V, *O, *dO;
  RowView qview, kview;            // Q, O, dO, dQ; K, V, dK, dV
  const float* LSE;                // [BH, nq]
  unsigned short *dQ, *dK, *dV;
  int nq, nk;                      // query rows, keys
  int nqblk, nkblk;                // blocks of 64
  int shift_blocks;                // causal: Q block i sees KV blocks j <= i + shift_blocks
  int k_smooth;
  float sm_scale, scale_log2e;
  int8_t *QF, *QT, *KF, *KT, *dOT; // the workspace's tensors
  float *sQ, *sK, *sdO, *delta, *nl2, *muK;
  int8_t* dSq;
  int ds_pitch;
  float* sdS;
};

template <int D, bool CAUSAL, int NB, bool SHARE>
__global__ void __launch_bounds__(512, 1) sage_bwd_short_kernel(ShortBwdArgs args) {
  typedef ShortBlock<D> Block;
  typedef typename Block::Raw Raw;
  typedef typename Block::Codes Codes;
  constexpr int KS = Block::KS, TILE = Block::TILE, EPT = Block::EPT, PER = Block::PER, SUMS = Block::SUMS;
  constexpr int PPR = D / 8;               // 16-byte pieces of a bf16 row
  constexpr int NTASK = SHARE ? NB : 3 * NB;       // blocks of dO, then of Q, of K
  struct Frags {                           // of the tiles [Q block][KV block]
    int8_t p[NB][NB][2][2][1024];          // [32 keys][32 queries]: psi(P), one key per lane
    int8_t ds[NB][NB][2][2][1024];         // psi(dS), one key per lane
    int8_t dst[NB][NB][2][2][1024];        // [32 queries][32 keys]: psi(dS), one query per lane
  };
  struct Lds {
    union {
      struct {
        int8_t qf[NB][TILE], kf[NB][TILE]; // F layouts
      };
      double sums[SHARE ? 1 : SUMS][D];       // (before them: of K)
      int8_t dq_rows[NB][2 * TILE];        // at the end: rows of a gradient, pieces as in dO
    };
    union {
      struct {
        int8_t qt[NB][TILE], kt[NB][TILE]; // TF layouts
      };
      unsigned raw[NB * TILE / 2];         // K as it came, for the sums
      int8_t dv_rows[NB][2 * TILE];
    };
    int8_t dot[NB][TILE];                  // psi(dO), TF layout
    union {
      struct {
        int8_t dof[NB][TILE];              // the same, F layout
        int8_t dO[NB][2 * TILE];           // bf16 dO, row by row; 16-byte piece c of row r in slot c ^ (r & (PPR - 1))
      };
      Frags f;
      int8_t dk_rows[NB][2 * TILE];
    };
    float nl2[64 * NB], dl[64 * NB];       // -L log2(e), -delta
    float red[NB][NB][4][2];               // [Q block][KV block][wave]: max P, max |dS|
    float amax[NTASK][8];
    float mu[D];
  };
  __shared__ __attribute__((aligned(16))) Lds L;

  const int bh = blockIdx.x;
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int ll = lane & 31, h = lane >> 5;
  const Block own(t);
  const int row = own.row;
  const int sb = CAUSAL ? args.shift_blocks : 0;

  // ---- loads: rows of dO and O (and Q and K), this wave's keys of V as operands of dP, or the codes ----
  Raw raw[NTASK], rawO[NB];
#pragma unroll
  for (int i = 0; i < NB; i++) {
    raw[i] = own.load(args.dO, args.qview, bh, i, args.nq);
    rawO[i] = own.load(args.O, args.qview, bh, i, args.nq);
  }
  if constexpr (!SHARE) {
#pragma unroll
    for (int i = 0; i < NB; i++) {
      raw[NB + i] = own.load(args.Q, args.qview, bh, i, args.nq);
      raw[2 * NB + i] = own.load(args.K, args.kview, bh, i, args.nk);
    }
  }
  const int jA = wave >> 2, kA = (wave >> 1) & 1, qA = wave & 1;      // S, dP, P, dS: KV block, 32 keys, 32 queries
  v8bf vfr[D / 16];
  {
    const int key = min(64 * jA + 32 * kA + ll, args.nk - 1);         // (a key that does not exist: its P is masked)
    const unsigned short* p = args.V + args.kview.row(bh, key) + 8 * h;
#pragma unroll
    for (int s = 0; s < D / 16; s++) vfr[s] = *(const v8bf*)(p + 16 * s);
  }
  if constexpr (SHARE) {
    // (all loads before the first store)
    constexpr int PIECES = (NB * TILE / 16 + 511) / 512;
    const int8_t* src[4] = {args.QF + (size_t)bh * args.nqblk * TILE, args.KF + (size_t)bh * args.nkblk * TILE,
                            args.QT + (size_t)bh * args.nqblk * TILE, args.KT + (size_t)bh * args.nkblk * TILE};
    int8_t* dst[4] = {L.qf[0], L.kf[0], L.qt[0], L.kt[0]};
    v4i piece[4][PIECES];
#pragma unroll
    for (int a = 0; a < 4; a++)
#pragma unroll
      for (int k = 0; k < PIECES; k++) {
        const int i = t + 512 * k, all = (a & 1 ? args.nkblk : args.nqblk) * (TILE / 16);
        piece[a][k] = *(const v4i*)(src[a] + 16 * min(i, all - 1));
      }
#pragma unroll
    for (int a = 0; a < 4; a++)
#pragma unroll
      for (int k = 0; k < PIECES; k++) {
        const int i = t + 512 * k, all = (a & 1 ? args.nkblk : args.nqblk) * (TILE / 16);
        if (i < all) *(v4i*)(dst[a] + 16 * i) = piece[a][k];
      }
  }
  float shared_scale = 0.f;                // lane k: s_Q of Q block k - NB, s_K of KV block k - 2 NB
  if constexpr (SHARE) {
    const int b = lane < 2 * NB ? min(max(lane - NB, 0), args.nqblk - 1) : min(lane < 3 * NB ? lane - 2 * NB : 0, args.nkblk - 1);
    shared_scale = lane < 2 * NB ? args.sQ[(size_t)bh * args.nqblk + b] : args.sK[(size_t)bh * args.nkblk + b];
  }
  if (t < 64 * NB && t < 64 * args.nqblk) {
    const float v = t < args.nq ? -args.LSE[(size_t)bh * args.nq + t] * 1.4426950408889634f : -INFINITY;
    L.nl2[t] = v;
    args.nl2[(size_t)bh * 64 * args.nqblk + t] = v;
  }

  // ---- delta = rowsum(dO o O), in the pre-pass's order: a row's 16-channel chunks, low and high eight in turn ----
#pragma unroll
  for (int i = 0; i < NB; i++) {
    float acc = 0.f;
    if constexpr (D == 128) {
#pragma unroll
      for (int e = 0; e < 8; e++) {
        acc += bf16_bits_to_float(raw[i][e]) * bf16_bits_to_float(rawO[i][e]);
        acc += bf16_bits_to_float(raw[i][8 + e]) * bf16_bits_to_float(rawO[i][8 + e]);
      }
    } else {
      // (a chunk is two threads here)
#pragma unroll
      for (int e = 0; e < 8; e++) {
        const float mine = bf16_bits_to_float(raw[i][e]) * bf16_bits_to_float(rawO[i][e]), other = __shfl_xor(mine, 1, 64);
        acc += t & 1 ? other : mine;
        acc += t & 1 ? mine : other;
      }
    }
#pragma unroll
    for (int off = D == 128 ? 1 : 2; off < 8; off <<= 1) acc += __shfl_xor(acc, off, 64);
    if ((t & 7) == 0 && i < args.nqblk) {
      L.dl[64 * i + row] = -acc;
      args.delta[((size_t)bh * args.nqblk + i) * 64 + row] = -acc;
    }
    // dO as it came, for dP
#pragma unroll
    for (int k = 0; k < EPT / 8; k++) {
      v8us v;
#pragma unroll
      for (int e = 0; e < 8; e++) v[e] = raw[i][8 * k + e];
      *(v8us*)(L.dO[i] + row * 2 * D + (((own.ch0 / 8 + k) ^ row) & (PPR - 1)) * 16) = v;
    }
  }

  // ---- psi of dO (and Q and K) ----
  float mu[EPT];
#pragma unroll
  for (int e = 0; e < EPT; e++) mu[e] = 0.f;
  if constexpr (!SHARE) {
    if (args.k_smooth) own.template mean<NB>(raw + 2 * NB, args.nkblk, args.nk, L.raw, L.sums, L.mu, args.muK + (size_t)bh * D, mu);
    else if (t < D) args.muK[(size_t)bh * D + t] = 0.f;
  }
  auto values = [&](int task, float (&x)[EPT]) __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < EPT; e++) {
      x[e] = bf16_bits_to_float(raw[task][e]);
      if (task >= 2 * NB) x[e] = 64 * (task - 2 * NB) + row < args.nk ? x[e] - mu[e] : 0.f;
    }
  };
#pragma unroll
  for (int k = 0; k < NTASK; k++) {
    float x[EPT], a = 0.f;
    values(k, x);
#pragma unroll
    for (int e = 0; e < EPT; e++) a = fmaxf(a, fabsf(x[e]));
    a = wave_max_nonneg_f32(a);
    if (lane == 0) L.amax[k][wave] = a;
  }
  __syncthreads();
  float scale, factor;                     // lane k has those of task k
  short_factors(L.amax[lane < NTASK ? lane : 0], scale, factor);
  const int f_at = own.f_at();
#pragma unroll
  for (int k = 0; k < NTASK; k++) {
    float x[EPT];
    values(k, x);
    const Codes c = Block::quantise(x, of_lane(factor, k));
    const int b = k % NB;
    *(Codes*)((k < NB ? L.dof[b] : k < 2 * NB ? L.qf[b] : L.kf[b]) + f_at) = c;
    if (k >= NB && k < 2 * NB && b < args.nqblk) *(Codes*)(args.QF + ((size_t)bh * args.nqblk + b) * TILE + f_at) = c;
    if (k >= 2 * NB && b < args.nkblk) *(Codes*)(args.KF + ((size_t)bh * args.nkblk + b) * TILE + f_at) = c;
  }
  if (wave == 0 && lane < NTASK) {
    const int b = lane % NB;
    if (lane < NB && b < args.nqblk) args.sdO[(size_t)bh * args.nqblk + b] = scale;
    if (lane >= NB && lane < 2 * NB && b < args.nqblk) args.sQ[(size_t)bh * args.nqblk + b] = scale;
    if (lane >= 2 * NB && b < args.nkblk) args.sK[(size_t)bh * args.nkblk + b] = scale;
  }
  __syncthreads();
  for (int i = t; i < NB * PER; i += 512) {
    const int b = i / PER;
    if (b < args.nqblk) Block::transpose(L.dof[b], i % PER, L.dot[b]);
    if constexpr (!SHARE) {
      if (b < args.nqblk) Block::transpose(L.qf[b], i % PER, L.qt[b]);
      if (b < args.nkblk) Block::transpose(L.kf[b], i % PER, L.kt[b]);
    }
  }
  __syncthreads();
  {
    auto leave = [&](const int8_t* src, int blocks, int8_t* dst) __attribute__((always_inline)) {
      int8_t* p = dst + (size_t)bh * blocks * TILE;
      for (int i = t; i < blocks * TILE / 16; i += 512) *(v4i*)(p + 16 * i) = *(const v4i*)(src + 16 * i);
    };
    leave(L.dot[0], args.nqblk, args.dOT);
    if constexpr (!SHARE) {
      leave(L.qt[0], args.nqblk, args.QT);
      leave(L.kt[0], args.nkblk, args.KT);
    }
  }

  // ---- S, dP, P, dS of all tiles, a quarter of each tile of its KV block a wave ----
  if constexpr (SHARE) scale = lane < NB ? scale : shared_scale;
  auto sd = [&](int i) __attribute__((always_inline)) { return of_lane(scale, i); };
  auto sq = [&](int i) __attribute__((always_inline)) { return of_lane(scale, NB + i); };
  auto sk = [&](int j) __attribute__((always_inline)) { return of_lane(scale, 2 * NB + j); };
  auto tile_exists = [&](int i, int j) __attribute__((always_inline)) { return i < args.nqblk && j < args.nkblk && (!CAUSAL || i + sb >= j); };
  const int jc = jA < NB ? jA : 0;                                           // (one block a head: waves 4 to 7 have no tile)
  float p[NB][16], ds[NB][16];
#pragma unroll
  for (int i = 0; i < NB; i++) {
    if (jA >= NB || !tile_exists(i, jA)) continue;
    v16i sacc;
    v16f dp;
#pragma unroll
    for (int r = 0; r < 16; r++) sacc[r] = 0;
#pragma unroll
    for (int s = 0; s < KS; s++)
      sacc = __builtin_amdgcn_mfma_i32_32x32x32_i8(*(const v4i*)(L.qf[i] + (qA * KS + s) * 1024 + lane * 16),
                                                   *(const v4i*)(L.kf[jc] + (kA * KS + s) * 1024 + lane * 16), sacc, 0, 0, 0);
    const float *nl = L.nl2 + 64 * i + 32 * qA + 4 * h, *dl = L.dl + 64 * i + 32 * qA + 4 * h;
#pragma unroll
    for (int r = 0; r < 16; r++) dp[r] = dl[8 * (r >> 2) + (r & 3)];
    const int8_t* rowp = L.dO[i] + (32 * qA + ll) * 2 * D;
#pragma unroll
    for (int s = 0; s < D / 16; s++)
      dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*(const v8bf*)(rowp + (((2 * s + h) ^ ll) & (PPR - 1)) * 16), vfr[s], dp, 0, 0, 0);
    const float c = sq(i) * sk(jc) * args.scale_log2e;
    const bool key_exists = 64 * jA + 32 * kA + ll < args.nk;
    const int diag = CAUSAL && i + sb == jA ? 32 * kA + ll : -1;             // the tile's queries before this one see not this key
    float pm = 0.f, dm = 0.f;
#pragma unroll
    for (int r = 0; r < 16; r++) {
      const float pv = __builtin_amdgcn_exp2f(__builtin_fmaf((float)sacc[r], c, nl[8 * (r >> 2) + (r & 3)]));
      p[i][r] = key_exists && 32 * qA + 8 * (r >> 2) + 4 * h + (r & 3) >= diag ? pv : 0.f;
      ds[i][r] = p[i][r] * dp[r];
      pm = fmaxf(pm, p[i][r]);
      dm = fmaxf(dm, fabsf(ds[i][r]));
    }
    pm = wave_max_nonneg_f32(pm);
    dm = wave_max_nonneg_f32(dm);
    if (lane == 0) {
      L.red[i][jc][wave & 3][0] = pm;
      L.red[i][jc][wave & 3][1] = dm;
    }
  }
  __syncthreads();
  // ---- psi(P), psi(dS) with the maxima of the tiles (see sage_bwd_wide_kernel: internal scales, 127 / a by rcp) ----
  auto tile_max = [&](int i, int j, int what) __attribute__((always_inline)) {
    return fmaxf(fmaxf(L.red[i][j][0][what], L.red[i][j][1][what]), fmaxf(L.red[i][j][2][what], L.red[i][j][3][what]));
  };
#pragma unroll
  for (int i = 0; i < NB; i++) {
    if (jA >= NB || !tile_exists(i, jA)) continue;
    const float bpm = tile_max(i, jc, 0), bdm = tile_max(i, jc, 1);
    const float rP = bpm > 0.f ? 127.0f * __builtin_amdgcn_rcpf(bpm) : 0.f;
    const float rS = bdm > 0.f ? 127.0f * __builtin_amdgcn_rcpf(bdm) : 0.f;
    v4i pf, df;
#pragma unroll
    for (int aa = 0; aa < 4; aa++) {
      unsigned up = 0, ub[4];
#pragma unroll
      for (int b = 0; b < 4; b++) {
        up = __builtin_amdgcn_cvt_pk_u8_f32(p[i][4 * aa + b] * rP, b, up);
        ub[b] = __float_as_uint(__builtin_fmaf(ds[i][4 * aa + b], rS, kRoundMagic));
      }
      pf[aa] = (int)up;
      df[aa] = (int)(__builtin_amdgcn_perm(ub[1], ub[0], 0x0c0c0400u) | __builtin_amdgcn_perm(ub[3], ub[2], 0x04000c0cu));
    }
    *(v4i*)(L.f.p[i][jc][kA][qA] + lane * 16) = pf;
    *(v4i*)(L.f.ds[i][jc][kA][qA] + lane * 16) = df;
    // byte (key ll, query 8 aa + 4 h + b) to lane (query, (key / 4) % 2), byte 4 (key / 8) + key % 4
    int8_t* tr = L.f.dst[i][jc][qA][kA] + 4 * h * 16 + ((ll >> 2) & 1) * 512 + 4 * (ll >> 3) + (ll & 3);
#pragma unroll
    for (int aa = 0; aa < 4; aa++)
#pragma unroll
      for (int b = 0; b < 4; b++) tr[(8 * aa + b) * 16] = (int8_t)(df[aa] >> (8 * b));
    const size_t tile = ((size_t)bh * args.nqblk + i) * args.ds_pitch + jA;
    *(v4i*)(args.dSq + tile * 4096 + qA * 2048 + kA * 1024 + lane * 16) = df;
    if (lane == 0) args.sdS[tile] = bdm * (1.0f / 127.0f);         // (the same value from all four)
  }
  __syncthreads();

  // A gradient leaves in whole rows: a wave's accumulators (one row per lane, 32 channels) go to LDS, and 16-byte pieces from there.
  // (As 8-byte pieces straight from the accumulators the stores of dV and dK alone took 4000 of 33000 cycles.)
  auto to_rows = [&](int first_row, int cb, const float (&x)[16], float factor, int8_t* rows) __attribute__((always_inline)) {
    const int r = first_row + ll;
    int8_t* out = rows + r * 2 * D + 8 * h;
#pragma unroll
    for (int aa = 0; aa < 4; aa++) {
      v4us o;
#pragma unroll
      for (int b = 0; b < 4; b++) o[b] = float_to_bf16_bits(x[4 * aa + b] * factor);
      *(v4us*)(out + (((4 * cb + aa) ^ r) & (PPR - 1)) * 16) = o;
    }
  };
  auto rows_out = [&](unsigned short* dst, const RowView& view, int n, const int8_t* rows) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < NB * 64 * PPR / 512; k++) {
      const int c = t + 512 * k, r = c / PPR, pc = c % PPR;
      if (r < n) *(v8us*)(dst + view.row(bh, r) + 8 * pc) = *(const v8us*)(rows + r * 2 * D + ((pc ^ r) & (PPR - 1)) * 16);
    }
  };

  // ---- dQ: 32 queries of each Q block, a channel block (d = 64: waves 0 to 3) ----
  const int qQ = wave / KS, cQ = wave % KS;
  if (qQ < 2) {
#pragma unroll
    for (int i = 0; i < NB; i++) {
      if (i >= args.nqblk) continue;
      float acc[16];
#pragma unroll
      for (int r = 0; r < 16; r++) acc[r] = 0.f;
#pragma unroll
      for (int j = 0; j < NB; j++) {
        if (!tile_exists(i, j)) continue;
        // (sums and weights as in sage_bwd_dq_kernel)
        v16i x = mfma_from_bias(*(const v4i*)(L.kt[j] + cQ * 1024 + lane * 16), *(const v4i*)(L.f.dst[i][j][qQ][0] + lane * 16));
        x = __builtin_amdgcn_mfma_i32_32x32x32_i8(*(const v4i*)(L.kt[j] + (KS + cQ) * 1024 + lane * 16), *(const v4i*)(L.f.dst[i][j][qQ][1] + lane * 16), x, 0, 0, 0);
        const float w = tile_max(i, j, 1) * (1.0f / 127.0f) * sk(j) * (args.sm_scale * kDqWeight);
#pragma unroll
        for (int r = 0; r < 16; r++) acc[r] = __builtin_fmaf(__int_as_float(x[r]) - kBiasC0, w, acc[r]);
      }
      to_rows(64 * i + 32 * qQ, cQ, acc, kDqWeight, L.dq_rows[0]);
    }
  }
  // ---- dV, dK: a channel block of one or two blocks of 32 keys ----
  constexpr int BKB = NB * KS == 8 ? 2 : 1;
  const int jB = NB == 2 ? wave >> 2 : 0, cB = wave % KS;
  const int kB = BKB == 2 ? 0 : NB == 2 ? (wave >> 1) & 1 : wave / KS;       // (one head of one block, d = 64: waves 4 to 7 have none)
  const bool hasB = kB < 2 && jB < args.nkblk;
  float dv[BKB][16], dk[BKB][16];
#pragma unroll
  for (int b = 0; b < BKB; b++)
#pragma unroll
    for (int r = 0; r < 16; r++) dv[b][r] = dk[b][r] = 0.f;
  if (hasB) {
#pragma unroll
    for (int i = NB - 1; i >= 0; i--) {
      if (!tile_exists(i, jB)) continue;
      const float sP = tile_max(i, jB, 0) * (1.0f / 127.0f), sS = tile_max(i, jB, 1) * (1.0f / 127.0f);
      const float w_dv = sP * sd(i), w_dk = sS * sq(i) * args.sm_scale;
#pragma unroll
      for (int b = 0; b < BKB; b++) {
        const int kb = BKB == 2 ? b : kB;
        v16i rv, rk;
#pragma unroll
        for (int r = 0; r < 16; r++) rv[r] = rk[r] = 0;
#pragma unroll
        for (int k = 0; k < 2; k++) {
          rv = __builtin_amdgcn_mfma_i32_32x32x32_i8(*(const v4i*)(L.dot[i] + (k * KS + cB) * 1024 + lane * 16), *(const v4i*)(L.f.p[i][jB][kb][k] + lane * 16), rv, 0, 0, 0);
          rk = __builtin_amdgcn_mfma_i32_32x32x32_i8(*(const v4i*)(L.qt[i] + (k * KS + cB) * 1024 + lane * 16), *(const v4i*)(L.f.ds[i][jB][kb][k] + lane * 16), rk, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 16; r++) {
          dv[b][r] = __builtin_fmaf((float)rv[r], w_dv, dv[b][r]);
          dk[b][r] = __builtin_fmaf((float)rk[r], w_dk, dk[b][r]);
        }
      }
    }
  }
  __syncthreads();
  rows_out(args.dQ, args.qview, args.nq, L.dq_rows[0]);
  if (hasB) {
#pragma unroll
    for (int b = 0; b < BKB; b++) {
      const int first_row = 64 * jB + 32 * (BKB == 2 ? b : kB);
      to_rows(first_row, cB, dv[b], 1.0f, L.dv_rows[0]);
      to_rows(first_row, cB, dk[b], 1.0f, L.dk_rows[0]);
    }
  }
  __syncthreads();
  rows_out(args.dV, args.kview, args.nk, L.dv_rows[0]);
  rows_out(args.dK, args.kview, args.nk, L.dk_rows[0]);
}

}  // namespace sage
