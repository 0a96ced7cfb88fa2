// Forward for short heads: psi and the attention in one launch.
//
// A call of a few short heads takes the time of its launches (about 4 us each, with the trips to memory that each begins and ends
// with), not of its work.  Here a workgroup of eight waves takes one Q block of a head with ALL keys of the head (at most KB blocks of
// 64): it sums K, quantises its Q block and every block of K and V, all 512 threads on a block together, and forms O from what lies in
// LDS then, with the arithmetic of sage_fwd_kernel, so that the bits are its (`converting`: with the converting path for all logits, as
// the decoding form has it; the sums in this form's order).  The blocks of a head are quantised by
// each of its Q blocks' workgroups; the one whose turn it is writes the codes to the workspace, where a backward or an inspection hook
// wants them.
//
// All rows are loaded before anything else and stay in registers as they came (8 registers a block at d = 128).  The sums of K go
// through LDS as the mean_inline form's do, in float64.  V^ (and for the workspace Q^ and K^) is turned from the F to the TF layout by
// 4 x 4 blocks of bytes, four 16-byte pieces of it per thread.  The attention is divided as in sage_fwd_quad_kernel, over all tiles at once.
#pragma once

#include "common.h"
#include "fwd_kernel.h"
#include "prepass_kernels.h"

namespace sage {

// (products and sums are rounded apart, as in the other forms, but where an FMA is written)
#pragma clang fp contract(off)

// In lane i of 32: a of lane i plus a of lane i + 32; in lane i + 32 the same of b.
__device__ __forceinline__ double sum_of_halves(double a, double b) {
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)__double2loint(a), (unsigned)__double2loint(b), false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)__double2hiint(a), (unsigned)__double2hiint(b), false, false);
  return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}

// What the kernels for short heads share: 512 threads on a block of 64 rows, eight to a row.
template <int D>
struct ShortBlock {
  static constexpr int KS = D / 32;
  static constexpr int TILE = 64 * D;                  // bytes of a block's codes
  static constexpr int EPT = TILE / 512;               // values per thread
  static constexpr int PER = TILE / 64;                // threads that turn a block from the F to the TF layout
  static constexpr int G = 2048 / D;                   // row groups of the column sums: a pair of channels of two of them per thread
  static constexpr int SUMS = 16;                      // of them or of pairs of them in LDS, four of a wave of the pre-pass
  typedef unsigned short Raw __attribute__((ext_vector_type(EPT)));
  typedef int Codes __attribute__((ext_vector_type(EPT / 4)));
  int row, ch0;                                        // this thread's row of every block, and its channels
  __device__ __forceinline__ ShortBlock(int t) : row(t >> 3), ch0((t & 7) * EPT) {}
  __device__ __forceinline__ Raw load(const unsigned short* src, const RowView& view, int bh, int blk, int rows) const {
    Raw r = {};
    const int n = 64 * blk + row;
    if (n < rows) {
      const unsigned short* p = src + view.row(bh, n) + ch0;
#pragma unroll
      for (int k = 0; k < EPT / 8; k++) {
        const v8us v = *(const v8us*)(p + 8 * k);
#pragma unroll
        for (int e = 0; e < 8; e++) r[8 * k + e] = v[e];
      }
    }
    return r;
  }
  // where the thread's codes lie in a block's F layout
  __device__ __forceinline__ int f_at() const {
    return (((row >> 5) * KS + ch0 / 32) * 64 + (row & 31) + 32 * ((ch0 >> 4) & 1)) * 16 + (ch0 & 15);
  }
  static __device__ __forceinline__ Codes quantise(const float (&x)[EPT], float r) {
    Codes c;
#pragma unroll
    for (int w = 0; w < EPT / 4; w++) c[w] = quantise_4(x[4 * w], x[4 * w + 1], x[4 * w + 2], x[4 * w + 3], r);
    return c;
  }
  // mu_K of the thread's channels: float64 sums, divided by N, rounded once to FP32 (rows that do not exist are zero in `raw`).  Barriers
  // inside; `rows_lds` (a bf16 image of the blocks) is free again behind it.  The sums are added in the order of the pre-pass: row groups as
  // the threads of column_sums have them, a wave's groups in pairs and pairs of pairs, then the waves in turn.  Sums of ordinary
  // data are exact in any order; where they are not (1e30 beside 1 in a channel), a forward and a backward of other forms still have
  // the same mean.
  template <int KB>
  __device__ __forceinline__ void mean(const Raw* raw, int nkblk, int nk, unsigned* rows_lds, double (*red)[D], float* mu_lds, float* mu_out,
                                       float (&mu)[EPT]) const {
    const int t = threadIdx.x;
#pragma unroll
    for (int j = 0; j < KB; j++) *(Raw*)((unsigned short*)rows_lds + (size_t)(64 * j + row) * D + ch0) = raw[j];
    __syncthreads();
    const int pair = t % (D / 2), g = t / (D / 2);
    double a0 = 0.0, a1 = 0.0, b0 = 0.0, b1 = 0.0;       // groups g and g + G / 2
    for (int r = g; r < 64 * nkblk; r += G) {
      const unsigned u = rows_lds[r * (D / 2) + pair], v = rows_lds[(r + G / 2) * (D / 2) + pair];
      a0 += (double)__uint_as_float(u << 16);
      a1 += (double)__uint_as_float(u & 0xffff0000u);
      b0 += (double)__uint_as_float(v << 16);
      b1 += (double)__uint_as_float(v & 0xffff0000u);
    }
    if constexpr (D == 64) {
      // (the halves of a wave hold a pair of groups: each adds one of its two pairs, so that half as many values go through LDS.  All 32 of
      // them there took registers that a fourth workgroup of a CU needs: 4096 heads of 64 39.0 -> 43.3 us)
      const int p = (g >> 1) + (t & 32 ? SUMS / 2 : 0);
      red[p][2 * pair] = sum_of_halves(a0, b0);
      red[p][2 * pair + 1] = sum_of_halves(a1, b1);
    } else {
      red[g][2 * pair] = a0;
      red[g][2 * pair + 1] = a1;
      red[g + G / 2][2 * pair] = b0;
      red[g + G / 2][2 * pair + 1] = b1;
    }
    __syncthreads();
    if (t < D) {
      double s = 0.0;
#pragma unroll
      for (int k = 0; k < SUMS; k += 4) {
        const double w = (red[k][t] + red[k + 1][t]) + (red[k + 2][t] + red[k + 3][t]);
        s = k == 0 ? w : s + w;
      }
      const float m = (float)(s / (double)nk);
      mu_lds[t] = m;
      if (mu_out != nullptr) mu_out[t] = m;
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < EPT; e += 4) {
      const v4f m = *(const v4f*)(mu_lds + ch0 + e);
#pragma unroll
      for (int k = 0; k < 4; k++) mu[e + k] = m[k];
    }
  }
  // F to TF layout: thread i of PER takes four channels of sixteen rows
  static __device__ __forceinline__ void transpose(const int8_t* f, int i, int8_t* out) {
    const int quad = i & 7, h = (i >> 3) & 1, cb = (i >> 4) % KS, rb = (i >> 4) / KS;
    const int c = 4 * quad;                              // channel 32 cb + c
    const int8_t* p = f + ((rb * KS + cb) * 64 + 32 * (c >> 4)) * 16 + (c & 15);
    v4i o[4];
#pragma unroll
    for (int a = 0; a < 4; a++) {
      unsigned r[4];
#pragma unroll
      for (int b = 0; b < 4; b++) r[b] = *(const unsigned*)(p + (8 * a + 4 * h + b) * 16);
      const unsigned t0 = __builtin_amdgcn_perm(r[1], r[0], 0x05010400u), t1 = __builtin_amdgcn_perm(r[1], r[0], 0x07030602u);
      const unsigned u0 = __builtin_amdgcn_perm(r[3], r[2], 0x05010400u), u1 = __builtin_amdgcn_perm(r[3], r[2], 0x07030602u);
      o[0][a] = (int)__builtin_amdgcn_perm(u0, t0, 0x05040100u);
      o[1][a] = (int)__builtin_amdgcn_perm(u0, t0, 0x07060302u);
      o[2][a] = (int)__builtin_amdgcn_perm(u1, t1, 0x05040100u);
      o[3][a] = (int)__builtin_amdgcn_perm(u1, t1, 0x07060302u);
    }
    int8_t* q = out + ((rb * KS + cb) * 64 + c + 32 * h) * 16;
#pragma unroll
    for (int k = 0; k < 4; k++) *(v4i*)(q + 16 * k) = o[k];
  }
};
// Scale and factor of psi from the maxima of eight waves.
__device__ __forceinline__ void short_factors(const float* p, float& scale, float& factor) {
  float a = p[0];
#pragma unroll
  for (int k = 1; k < 8; k++) a = fmaxf(a, p[k]);
  const bool nz = a > 0.f;
  scale = nz ? a / 127.0f : 0.f;
  factor = nz ? 127.0f / a : 0.f;
}
__device__ __forceinline__ float of_lane(float v, int lane) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane)); }

struct ShortArgs {
  const unsigned short *Q, *K, *V;
  RowView qview, kview;            // Q and O; K and V
  unsigned short* O;
  float* LSE;                      // [BH, nq]
  int nq, nk;                      // query rows, keys
  int nqblk, nkblk;                // blocks of 64
  int shift;                       // causal: query i sees keys k <= i + shift
  int heads, own_xcd;              // see prepass_item
  int k_smooth;
  int converting;                  // the logits by the converting path whatever their scales (see fwd_short_impl)
  float scale_log2e;
  // the workspace's tensors, or nullptr (TF layouts of Q and K: where a backward shares them)
  int8_t *QF, *QT, *KF, *KT, *VT;
  float *sQ, *sK, *sV, *muK;
};

template <int D, bool CAUSAL, int KB>
__global__ void __launch_bounds__(512, 1) sage_fwd_short_kernel(ShortArgs args) {
  typedef ShortBlock<D> Block;
  constexpr int KS = Block::KS, TILE = Block::TILE, EPT = Block::EPT, PER = Block::PER, SUMS = Block::SUMS;
  constexpr int NTASK = 2 * KB + 1;        // blocks of K, of V, the one of Q
  struct Lds {
    int8_t kf[KB][TILE];                   // K^, F layout
    int8_t qf[TILE];                       // Q^, F layout
    union {
      struct {
        int8_t vf[KB][TILE];               // V^, F layout
        int8_t vt[KB][TILE];               // V^, TF layout
      };
      unsigned raw[KB * TILE / 2];         // K as it came, for the sums
    };
    float mu[D];
    float amax[NTASK][8];                  // maxima of the eight waves
    union {
      double red[SUMS][D];
      struct {
        int8_t p[2][KB][2][1024];          // [32 queries][tile][32 keys]: P^, the operand of P^V^
        float psum[2][KB][2][64];          // sums of P
        int rmax[2][KB][2][32];            // row maxima of the logits
      };
    };
  };
  __shared__ __attribute__((aligned(16))) Lds L;

  const PrepassItem item = prepass_item(blockIdx.x, blockIdx.y, blockIdx.z, args.own_xcd != 0, args.heads);
  const int bh = item.head, qb = item.block;
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const Block own(t);
  const int row = own.row;

  typename Block::Raw raw[NTASK];
#pragma unroll
  for (int j = 0; j < KB; j++) raw[j] = own.load(args.K, args.kview, bh, j, args.nk);
#pragma unroll
  for (int j = 0; j < KB; j++) raw[KB + j] = own.load(args.V, args.kview, bh, j, args.nk);
  raw[2 * KB] = own.load(args.Q, args.qview, bh, qb, args.nq);

  float mu[EPT];
#pragma unroll
  for (int e = 0; e < EPT; e++) mu[e] = 0.f;
  float* mu_out = args.muK != nullptr && qb == 0 ? args.muK + (size_t)bh * D : nullptr;
  if (args.k_smooth) own.template mean<KB>(raw, args.nkblk, args.nk, L.raw, L.red, L.mu, mu_out, mu);
  else if (mu_out != nullptr && t < D) mu_out[t] = 0.f;

  // ---- psi: block maxima, scales, codes ----
  auto values = [&](int task, float (&x)[EPT]) __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < EPT; e++) {
      x[e] = bf16_bits_to_float(raw[task][e]);
      if (task < KB) x[e] = 64 * task + row < args.nk ? x[e] - mu[e] : 0.f;      // (rows that do not exist are zero behind the smoothing)
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
  // lane k has the factors of task k
  float scale, factor;
  short_factors(L.amax[lane < NTASK ? lane : 0], scale, factor);
  auto of_task = [](float v, int task) __attribute__((always_inline)) { return of_lane(v, task); };
  const int f_at = own.f_at();
  const bool writes = args.QF != nullptr;
  auto my_turn = [&](int j) { return writes && j < args.nkblk && j % args.nqblk == qb; };
  typedef typename Block::Codes Codes;
#pragma unroll
  for (int k = 0; k < NTASK; k++) {
    float x[EPT];
    values(k, x);
    const Codes c = Block::quantise(x, of_task(factor, k));
    int8_t* f = k < KB ? L.kf[k] : k < 2 * KB ? L.vf[k - KB] : L.qf;
    *(Codes*)(f + f_at) = c;
    if (k < KB && my_turn(k)) *(Codes*)(args.KF + ((size_t)bh * args.nkblk + k) * TILE + f_at) = c;
    if (k == 2 * KB && writes) *(Codes*)(args.QF + ((size_t)bh * args.nqblk + qb) * TILE + f_at) = c;
  }
  if (writes && wave == 7) {
    if (lane < KB && my_turn(lane)) args.sK[(size_t)bh * args.nkblk + lane] = scale;
    if (lane >= KB && lane < 2 * KB && my_turn(lane - KB)) args.sV[(size_t)bh * args.nkblk + lane - KB] = scale;
    if (lane == 2 * KB) args.sQ[(size_t)bh * args.nqblk + qb] = scale;
  }
  __syncthreads();

  for (int i = t; i < KB * PER; i += 512) {
    const int j = i / PER;
    if (j < args.nkblk) Block::transpose(L.vf[j], i % PER, L.vt[j]);
  }
  // ---- the attention.  Four waves share 32 queries: wave (jj, kb) has 32-key block kb of the tiles jj, jj + 2, ... for the logits and P,
  // and channel block 2 jj + kb for O.  Row maxima, P^ and the sums of P go through LDS; every value is formed as in fwd_tile, and
  // the tiles are added in their order. ----
  const int ql = lane & 31, h = lane >> 5;
  const int qg = wave >> 2, jj = (wave >> 1) & 1, kb = wave & 1;
  const int q0 = 64 * qb + 32 * qg, q = q0 + ql;
  const int qlim = CAUSAL ? q + args.shift : args.nk - 1;
  const int last = CAUSAL ? (q0 + 31 + args.shift) / kBlock : args.nkblk - 1;
  constexpr int OWN = (KB + 1) / 2;                      // tiles of a wave
  const float cq = of_task(scale, 2 * KB) * args.scale_log2e;
  float smax = 0.f;
#pragma unroll
  for (int j = 0; j < KB; j++)
    if (j <= last) smax = fmaxf(smax, of_task(scale, j));
  auto attend = [&](auto sbias_tag) __attribute__((always_inline)) {
    constexpr bool SBIAS = decltype(sbias_tag)::value;
    v16i sacc[OWN];
    {
      v4i qf[KS];
#pragma unroll
      for (int s = 0; s < KS; s++) qf[s] = *(const v4i*)(L.qf + (qg * KS + s) * 1024 + lane * 16);
#pragma unroll
      for (int o = 0; o < OWN; o++) {
        const int j = jj + 2 * o;
        if (j > last) continue;
        const int8_t* k = L.kf[j] + kb * KS * 1024 + lane * 16;
        v16i zero;
#pragma unroll
        for (int r = 0; r < 16; r++) zero[r] = 0;
        if constexpr (SBIAS) sacc[o] = mfma_from_bias(*(const v4i*)k, qf[0]);
        else sacc[o] = __builtin_amdgcn_mfma_i32_32x32x32_i8(*(const v4i*)k, qf[0], zero, 0, 0, 0);
#pragma unroll
        for (int s = 1; s < KS; s++) sacc[o] = __builtin_amdgcn_mfma_i32_32x32x32_i8(*(const v4i*)(k + s * 1024), qf[s], sacc[o], 0, 0, 0);
        int m = INT_MIN;
#pragma unroll
        for (int r = 0; r < 16; r++) {
          const int key = j * kBlock + 32 * kb + 8 * (r >> 2) + 4 * h + (r & 3);
          sacc[o][r] = key > qlim ? INT_MIN : sacc[o][r];
          m = max(m, sacc[o][r]);
        }
        m = half_swap_max_i32(m);
        if (h == 0) L.rmax[qg][j][kb][ql] = m;
      }
    }
    __syncthreads();
    // the running reference behind each tile, and each tile's weight against it (alpha: 1 where it was not raised)
    float m_ref = -INFINITY, alpha[KB], beta[KB], off[KB];
#pragma unroll
    for (int j = 0; j < KB; j++) {
      if (j > last) break;
      const float c = cq * of_task(scale, j);
      const int mrow = max(L.rmax[qg][j][0][ql], L.rmax[qg][j][1][ql]);
      const float mloc = (float)(mrow - (SBIAS ? kBiasBits : 0)) * c;
      alpha[j] = 1.f;
      if (__builtin_amdgcn_ballot_w64(mloc > m_ref + kTau) != 0) {
        const float m_new = fmaxf(m_ref, mloc);
        alpha[j] = __builtin_amdgcn_exp2f(m_ref - m_new);
        m_ref = m_new;
      }
      beta[j] = __builtin_amdgcn_exp2f(mloc - m_ref);
      off[j] = SBIAS ? __builtin_fmaf(-__int_as_float(mrow), c * kTwo26, kLog2_127) : kLog2_127 - mloc;
    }
#pragma unroll
    for (int o = 0; o < OWN; o++) {
      const int j = jj + 2 * o;
      if (j > last) continue;
      const float c = cq * of_task(scale, j), c_eff = SBIAS ? c * kTwo26 : c;
      const float offj = jj == 0 ? off[2 * o] : off[2 * o + 1 < KB ? 2 * o + 1 : 0];
      float psum[4] = {0.f, 0.f, 0.f, 0.f};
      v4i pf;
#pragma unroll
      for (int aa = 0; aa < 4; aa++) {
        unsigned u = 0;
#pragma unroll
        for (int b = 0; b < 4; b++) {
          const int sv = sacc[o][4 * aa + b];
          float x = __builtin_fmaf(SBIAS ? __int_as_float(sv) : (float)sv, c_eff, offj);
          x = sv == INT_MIN ? -INFINITY : x;
          const float e = __builtin_amdgcn_exp2f(x);
          psum[b] = aa == 0 ? e : psum[b] + e;
          u = __builtin_amdgcn_cvt_pk_u8_f32(e, b, u);
        }
        pf[aa] = (int)u;
      }
      *(v4i*)(L.p[qg][j][kb] + lane * 16) = pf;
      L.psum[qg][j][kb][lane] = (psum[0] + psum[1]) + (psum[2] + psum[3]);
    }
    __syncthreads();
    const int cb = 2 * jj + kb;
    if (cb >= KS) return;
    float l_part[2] = {0.f, 0.f}, w_bias = 0.f, oacc[16];
#pragma unroll
    for (int r = 0; r < 16; r++) oacc[r] = 0.f;
#pragma unroll
    for (int j = 0; j < KB; j++) {
      if (j > last) break;
      const int8_t* v = L.vt[j] + cb * 1024 + lane * 16;
      v16i tt = mfma_from_bias(*(const v4i*)v, *(const v4i*)(L.p[qg][j][0] + lane * 16));
      tt = __builtin_amdgcn_mfma_i32_32x32x32_i8(*(const v4i*)(v + KS * 1024), *(const v4i*)(L.p[qg][j][1] + lane * 16), tt, 0, 0, 0);
      const float w = beta[j] * of_task(scale, KB + j) * kTwo26;
#pragma unroll
      for (int k = 0; k < 2; k++) l_part[k] = __builtin_fmaf(beta[j], L.psum[qg][j][k][lane], j == 0 ? 0.f : l_part[k] * alpha[j]);
      w_bias = j == 0 ? w : w_bias * alpha[j] + w;
#pragma unroll
      for (int r = 0; r < 16; r++) oacc[r] = __builtin_fmaf(__int_as_float(tt[r]), w, j == 0 ? 0.f : oacc[r] * alpha[j]);
    }
    const float corr = kBiasC0 * w_bias;
    const float l_tot = half_swap_sum_f32(l_part[0]) + half_swap_sum_f32(l_part[1]);
    const float inv_l = 1.0f / l_tot;
    if (q >= args.nq) return;
    unsigned short* Oh = args.O + args.qview.row(bh, q) + 32 * cb + 4 * h;
#pragma unroll
    for (int aa = 0; aa < 4; aa++) {
      v4us o;
#pragma unroll
      for (int b = 0; b < 4; b++) o[b] = float_to_bf16_bits((oacc[4 * aa + b] - corr) * inv_l);
      *(v4us*)(Oh + 8 * aa) = o;
    }
    if (cb == 0 && h == 0) args.LSE[(size_t)bh * args.nq + q] = (m_ref + __builtin_amdgcn_logf(l_tot) - kLog2_127) * kLn2;
  };
  static_assert(KB < kBiasPeriod, "the bias is subtracted once, at the end");
  // (see sage_fwd_kernel for the line)
  if (__builtin_amdgcn_readfirstlane((int)(!args.converting && cq * smax < 1e-3f))) attend(std::true_type{});
  else attend(std::false_type{});
  if (!writes) return;
  for (int j = 0; j < args.nkblk; j++) {
    if (!my_turn(j)) continue;
    if (args.KT != nullptr && t < PER) Block::transpose(L.kf[j], t, args.KT + ((size_t)bh * args.nkblk + j) * TILE);
    int8_t* out = args.VT + ((size_t)bh * args.nkblk + j) * TILE;
    for (int i = t; i < TILE / 16; i += 512) *(v4i*)(out + 16 * i) = *(const v4i*)(L.vt[j] + 16 * i);
  }
  if (args.QT != nullptr && t >= 512 - PER) Block::transpose(L.qf, t - (512 - PER), args.QT + ((size_t)bh * args.nqblk + qb) * TILE);
}

}  // namespace sage
