// Forward for at most 32 query rows per head that see every key (a decoding step against a cache).
//
// Such a call is bound by reading K and V: the products are nothing, and every key is used once, so
// quantising K and V into a workspace and reading the codes back costs more than the rest together (two query
// sequences of 32 heads against 8192 keys, d = 128: 109 us of pre-pass and 167 us of forward, the latter on 64
// workgroups, where one pass over the 268 MB of K and V takes about 55 us at the rate of a large copy).  Here a
// wave takes whole 64-key blocks straight from the caller's tensors: it loads a block of K in the order of
// the F fragments, finds the block's scale, quantises in registers, forms the logits, and does the same with V,
// whose fragments one MFMA against the identity turns from (lane = key) to (lane = channel), the operand form of
// P^V^.  No barrier and no traffic but K and V inside the loop (and at d = 128 two fragments of psi(Q) from LDS).  psi is the
// pre-pass's function (quantise_16, clamp and factor included), so codes and scales are the same bits for every input, NaN and
// blocks whose 127 / max|x| overflows among them; the logits are formed as in sage_fwd_kernel's converting path.
//
// Keys are split over waves (four to a workgroup, which meet in LDS) and workgroups (whose partial O, m, l a second
// small kernel joins).
//
// Two waves to a SIMD.  A wave alone gets a vector instruction out every 4.8 cycles and a block took it about 2800, so one
// wave per SIMD, with K and V both loaded a block ahead, was bound by issue as much as by memory (two sequences of 32 heads of
// 8192 keys: 65 us of the call's 92).  For d = 128 two waves have room for one block of raw values each: V is loaded under the
// logits into the registers that K has left, the next K under P^V^, values are formed twice (for the maximum and for
// the codes) and not held, and lane-derived values are recomputed.  The call 92.4 -> 82.8 us (with the join below; 79.1 since no
// block is read twice); 8 sequences of 32 heads of 4096 159 -> 148; 32 heads of 8192, d = 64, 16 queries, four sequences 87 -> 75.
#pragma once

#include "common.h"
#include "fwd_kernel.h"
#include "prepass_kernels.h"

namespace sage {

struct DecodeArgs {
  const unsigned short *Q, *K, *V;
  RowView qview, kview;        // Q and O; K and V
  const double* mean_part;     // K-smoothing: float64 column sums [BH, nchunk, D] or nullptr
  int nchunk;
  unsigned short* O;
  float* LSE;                  // [BH, nq]
  float* part;                 // partial O of every workgroup [BH, nsplit, 32, D] (rows < nq used), if more than one
  v2f* part_ml;                // (m, l) [BH, nsplit, 32]
  int nq, nk, nblk;            // query rows (<= 32), keys, key blocks
  int blocks_per_wave;
  int nsplit;                  // workgroups of a head
  int heads;
  float scale_log2e;
};

template <int D, bool KSMOOTH, bool OWN_XCD = false>
__global__ void __launch_bounds__(256, 2) sage_fwd_decode_kernel(DecodeArgs args) {
  constexpr int KS = D / 32;
  constexpr int Q_LDS = D == 128 ? 2 : 0;    // fragments of psi(Q), the same for all four waves, that lie in LDS: nothing is in scratch then
  constexpr bool V_AHEAD = D == 64;          // registers for K and V a block ahead, in two waves per SIMD
  __shared__ __attribute__((aligned(16))) float mu_s[D];
  __shared__ __attribute__((aligned(16))) float xch[4 * KS * 4 * 64 * 4];    // partial O of the four waves
  __shared__ v2f ml[4 * 32];
  __shared__ v4i q_lds[Q_LDS ? 64 * Q_LDS : 1];                               // the last fragments of psi(Q)
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int r32 = lane & 31, h = lane >> 5;
  const PrepassItem item = prepass_item(blockIdx.x, blockIdx.y, blockIdx.z, OWN_XCD, args.heads);
  const int bh = item.head, split = item.block;

  // this wave's fragments of a block: row 32 rb + r32, channels 32 s + 16 h .. + 16 (two 16-byte pieces)
  struct Raw {
    v8us v[2][KS][2];
  };
  auto load_block = [&](const unsigned short* src, const int j, const bool mine, const int r32, const int h, Raw& x) __attribute__((always_inline)) {
#pragma unroll
    for (int rb = 0; rb < 2; rb++) {
      const int row = decode_row(64 * j + 32 * rb + r32, mine, args.nk);
      const unsigned short* p = src + args.kview.row(bh, row) + 16 * h;
#pragma unroll
      for (int s = 0; s < KS; s++) {
        x.v[rb][s][0] = *(const v8us*)(p + 32 * s);
        x.v[rb][s][1] = *(const v8us*)(p + 32 * s + 8);
      }
    }
  };
  // Values of one fragment (K: minus the mean).  A row that does not exist holds the last one that does, which changes no
  // maximum of its block; its key is masked, its query not stored.
  auto values = [&](auto with_mean, const v8us (&raw)[2], const float* mu, float (&x)[16]) __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < 16; e++) x[e] = bf16_bits_to_float(raw[e >> 3][e & 7]);
    if constexpr (decltype(with_mean)::value) {
#pragma unroll
      for (int w = 0; w < 4; w++) {
        const v4f m = *(const v4f*)(mu + 4 * w);
#pragma unroll
        for (int e = 0; e < 4; e++) x[4 * w + e] = x[4 * w + e] - m[e];
      }
    }
  };
  // Codes of a block as F fragments; returns the block's scale.  At d = 64 blocks of ordinary numbers are left unclamped: no x * r is
  // further than 127 (1 + 2^-22) from zero.  Their maximum is formed with v_maximum3_f32, which keeps a NaN and so tells of one; a
  // block with NaN or infinities or of the smallest numbers takes the maximum without NaN and the clamp.  Whole calls, us, clamped -> not:
  // 128 heads of 2048 keys 27.95 -> 27.21, 4096 42.14 -> 41.46, 32 rows against 8192 75.64 -> 75.19, 16 of 20000 34.29 -> 33.92.  At d = 128
  // the second form of the block takes registers from the first, and memory is what it waits for (64 heads of 8192 70.4 both).
  auto quantise_block = [&](auto with_mean, Raw& raw, const int h, v4i (&f)[2][KS]) __attribute__((always_inline)) {
    int mu_at = 16 * h;
    // (the values are formed anew each time rather than held: raw, they take half the registers)
    auto anew = [&]() __attribute__((always_inline)) {
      asm volatile("" : "+v"(mu_at));
#pragma unroll
      for (int rb = 0; rb < 2; rb++)
#pragma unroll
        for (int s = 0; s < KS; s++) asm volatile("" : "+v"(raw.v[rb][s][0]), "+v"(raw.v[rb][s][1]));
    };
    auto block_max = [&](auto keeps_nan) __attribute__((always_inline)) {
      float a = 0.f;
#pragma unroll
      for (int s = 0; s < KS; s++) {
#pragma unroll
        for (int rb = 0; rb < 2; rb++) {
          float x[16];
          values(with_mean, raw.v[rb][s], mu_s + 32 * s + mu_at, x);
#pragma unroll
          for (int e = 0; e < 16; e++) a = decltype(keeps_nan)::value ? __builtin_elementwise_maximum(a, fabsf(x[e])) : fmaxf(a, fabsf(x[e]));
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      return wave_max_nonneg_f32(a);
    };
    auto codes = [&](auto clamp, const float r) __attribute__((always_inline)) {
#pragma unroll
      for (int s = 0; s < KS; s++) {
#pragma unroll
        for (int rb = 0; rb < 2; rb++) {
          float x[16];
          values(with_mean, raw.v[rb][s], mu_s + 32 * s + mu_at, x);
          f[rb][s] = quantise_16<decltype(clamp)::value>(x, r);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    asm volatile("" : "+v"(mu_at));
    float a;
    if constexpr (D == 64) {
      a = block_max(std::true_type{});
      anew();
      if (__builtin_amdgcn_readfirstlane((int)((a >= 1e-30f && a <= 3e38f) || a == 0.f))) {
        codes(std::false_type{}, a > 0.f ? 127.0f / a : 0.f);
        return a / 127.0f;
      }
      anew();
    }
    a = block_max(std::false_type{});
    anew();
    const bool nz = a > 0.f;
    codes(std::true_type{}, nz ? 127.0f / a : 0.f);
    return nz ? a / 127.0f : 0.f;
  };

  const int first = (split * 4 + wave) * args.blocks_per_wave;
  const int end = min(first + args.blocks_per_wave, args.nblk);
  Raw kr, vr_ahead;
  Raw& vr = V_AHEAD ? vr_ahead : kr;
  load_block(args.K, first, first < end, r32, h, kr);
  if constexpr (V_AHEAD) load_block(args.V, first, first < end, r32, h, vr);

  // psi(Q): the rows of the one query block
  v4i qf[KS];
  float cq;
  {
    float a = 0.f;
    v8us raw[KS][2];
    const unsigned short* p = args.Q + args.qview.row(bh, min(r32, args.nq - 1)) + 16 * h;
#pragma unroll
    for (int s = 0; s < KS; s++) {
      raw[s][0] = *(const v8us*)(p + 32 * s);
      raw[s][1] = *(const v8us*)(p + 32 * s + 8);
    }
#pragma unroll
    for (int s = 0; s < KS; s++) {
      float x[16];
      values(std::false_type{}, raw[s], nullptr, x);
#pragma unroll
      for (int e = 0; e < 16; e++) a = fmaxf(a, fabsf(x[e]));
    }
    a = wave_max_nonneg_f32(a);
    const bool nz = a > 0.f;
    const float r = nz ? 127.0f / a : 0.f;
#pragma unroll
    for (int s = 0; s < KS; s++) {
      float x[16];
      values(std::false_type{}, raw[s], nullptr, x);
      qf[s] = quantise_16(x, r);
    }
    cq = (nz ? a / 127.0f : 0.f) * args.scale_log2e;
  }
  // (every wave writes the same values and reads only after its own writes)
#pragma unroll
  for (int s = 0; s < Q_LDS; s++) q_lds[64 * s + lane] = qf[KS - Q_LDS + s];
  if constexpr (KSMOOTH) {
    // mu_K as prepass_quant_kernel forms it: chunk sums added in float64 in the same order, divided by N, rounded once to FP32
    double* red = (double*)xch;
    head_sums<D>(args.mean_part + (size_t)bh * args.nchunk * D, args.nchunk, red);
    if (t < D) {
      double s = red[t];
#pragma unroll
      for (int g = 1; g < 256 / D; g++) s += red[g * D + t];
      mu_s[t] = (float)(s / (double)args.nk);
    }
    __syncthreads();
  }

  // identity as the B operand of the transposing MFMA: lane (n, hh) holds k = 16 hh + t in byte t
  v4i ident;
#pragma unroll
  for (int w = 0; w < 4; w++) {
    unsigned u = 0;
#pragma unroll
    for (int e = 0; e < 4; e++) u |= (unsigned)((16 * h + 4 * w + e) == r32) << (8 * e);
    ident[w] = (int)u;
  }

  float oacc[KS][16];
#pragma unroll
  for (int cb = 0; cb < KS; cb++)
#pragma unroll
    for (int r = 0; r < 16; r++) oacc[cb][r] = 0.f;
  float w_bias = 0.f, m_ref = -INFINITY, l_part = 0.f;
  auto unbias = [&]() __attribute__((always_inline)) {
    const float corr = kBiasC0 * w_bias;
#pragma unroll
    for (int cb = 0; cb < KS; cb++)
#pragma unroll
      for (int r = 0; r < 16; r++) oacc[cb][r] -= corr;
    w_bias = 0.f;
  };

  // counted anew for each block and behind the loop, so that nothing derived from it holds a register through it
  auto lane_anew = []() __attribute__((always_inline)) {
    int zero = 0;
    asm volatile("" : "+s"(zero));
    return (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, zero));
  };
  for (int j = first; j < end; j++) {
    const int ln = lane_anew(), r32 = ln & 31, h = ln >> 5;
    v4i f[2][KS];
    const float sk = quantise_block(std::integral_constant<bool, KSMOOTH>{}, kr, h, f);
    const bool more = j + 1 < end;
    if constexpr (V_AHEAD) load_block(args.K, j + 1, more, r32, h, kr);       // what comes next travels under this block's arithmetic
    else load_block(args.V, j, true, r32, h, vr);
    __builtin_amdgcn_sched_barrier(0);
    v16i sacc[2];
#pragma unroll
    for (int s = 0; s < Q_LDS; s++) qf[KS - Q_LDS + s] = q_lds[64 * s + ln];
#pragma unroll
    for (int kb = 0; kb < 2; kb++) {
#pragma unroll
      for (int r = 0; r < 16; r++) sacc[kb][r] = 0;
#pragma unroll
      for (int s = 0; s < KS; s++) sacc[kb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(f[kb][s], qf[s], sacc[kb], 0, 0, 0);
    }
    const float c = cq * sk;
    // keys that do not exist: only the last block of a head has any (masking every block was 128 of its 2800 instructions: 128
    // heads of 2048 keys, d = 64, 29.5 -> 28.4 us; 64 of 8192, d = 128, 82.6 -> 81.9)
    const bool ragged = 64 * j + 64 > args.nk;
    auto exists = [&](const int kb, const int r) __attribute__((always_inline)) {
      return 64 * j + 32 * kb + 8 * (r >> 2) + 4 * h + (r & 3) < args.nk;
    };
    if (ragged) {
#pragma unroll
      for (int kb = 0; kb < 2; kb++)
#pragma unroll
        for (int r = 0; r < 16; r++) sacc[kb][r] = exists(kb, r) ? sacc[kb][r] : INT_MIN;
    }
    int mi[2] = {INT_MIN, INT_MIN};
#pragma unroll
    for (int kb = 0; kb < 2; kb++)
#pragma unroll
      for (int r = 0; r < 16; r++) mi[kb] = max(mi[kb], sacc[kb][r]);
    const float mloc = (float)half_swap_max_i32(max(mi[0], mi[1])) * c;
    if (__builtin_amdgcn_ballot_w64(mloc > m_ref + kTau) != 0) {
      const float m_new = fmaxf(m_ref, mloc);
      const float alpha = __builtin_amdgcn_exp2f(m_ref - m_new);
      l_part *= alpha;
      w_bias *= alpha;
#pragma unroll
      for (int cb = 0; cb < KS; cb++)
#pragma unroll
        for (int r = 0; r < 16; r++) oacc[cb][r] *= alpha;
      m_ref = m_new;
    }
    const float beta = __builtin_amdgcn_exp2f(mloc - m_ref);
    const float off = kLog2_127 - mloc;
    float xv[2][16];
#pragma unroll
    for (int kb = 0; kb < 2; kb++)
#pragma unroll
      for (int r = 0; r < 16; r++) xv[kb][r] = __builtin_fmaf((float)sacc[kb][r], c, off);
    if (ragged) {
#pragma unroll
      for (int kb = 0; kb < 2; kb++)
#pragma unroll
        for (int r = 0; r < 16; r++) xv[kb][r] = exists(kb, r) ? xv[kb][r] : -INFINITY;
    }
    float psum[4] = {0.f, 0.f, 0.f, 0.f};
    v4i pf[2];
#pragma unroll
    for (int kb = 0; kb < 2; kb++)
#pragma unroll
      for (int aa = 0; aa < 4; aa++) {
        unsigned u = 0;
#pragma unroll
        for (int b = 0; b < 4; b++) {
          const float e = __builtin_amdgcn_exp2f(xv[kb][4 * aa + b]);
          psum[b] += e;
          u = __builtin_amdgcn_cvt_pk_u8_f32(e, b, u);
        }
        pf[kb][aa] = (int)u;
      }
    l_part = __builtin_fmaf(beta, (psum[0] + psum[1]) + (psum[2] + psum[3]), l_part);
    __builtin_amdgcn_sched_barrier(0);
    const float sv = quantise_block(std::false_type{}, vr, h, f);
    if constexpr (V_AHEAD) load_block(args.V, j + 1, more, r32, h, vr);
    else load_block(args.K, j + 1, more, r32, h, kr);
    __builtin_amdgcn_sched_barrier(0);
    const float w = beta * sv * kTwo26;
    w_bias += w;
#pragma unroll
    for (int cb = 0; cb < KS; cb++) {
      v16i tt;
#pragma unroll
      for (int kb = 0; kb < 2; kb++) {
        v16i z;
#pragma unroll
        for (int r = 0; r < 16; r++) z[r] = 0;
        const v16i tr = __builtin_amdgcn_mfma_i32_32x32x32_i8(f[kb][cb], ident, z, 0, 0, 0);
        v4i va;
#pragma unroll
        for (int aa = 0; aa < 4; aa++)
          va[aa] = (int)(__builtin_amdgcn_perm((unsigned)tr[4 * aa + 1], (unsigned)tr[4 * aa], 0x0c0c0400u) |
                         __builtin_amdgcn_perm((unsigned)tr[4 * aa + 3], (unsigned)tr[4 * aa + 2], 0x04000c0cu));
        if (kb == 0) tt = mfma_from_bias(va, pf[kb]);
        else tt = __builtin_amdgcn_mfma_i32_32x32x32_i8(va, pf[kb], tt, 0, 0, 0);
      }
#pragma unroll
      for (int r = 0; r < 16; r++) oacc[cb][r] = __builtin_fmaf(__int_as_float(tt[r]), w, oacc[cb][r]);
      if (cb & 1) __builtin_amdgcn_sched_barrier(0);
    }
    if (((j - first) & (kBiasPeriod - 1)) == kBiasPeriod - 1) unbias();
  }
  unbias();

  // ---- the four waves meet: wave s finishes channel block s ----
  const int ln = lane_anew(), row = ln & 31, half = ln >> 5;
  const float l_tot = half_swap_sum_f32(l_part);
#pragma unroll
  for (int cb = 0; cb < KS; cb++)
#pragma unroll
    for (int aa = 0; aa < 4; aa++)
      *(v4f*)(xch + (((wave * KS + cb) * 4 + aa) * 64 + ln) * 4) =
          v4f{oacc[cb][4 * aa], oacc[cb][4 * aa + 1], oacc[cb][4 * aa + 2], oacc[cb][4 * aa + 3]};
  if (half == 0) ml[wave * 32 + row] = v2f{m_ref, l_tot};
  __syncthreads();
  if (row >= args.nq) return;
  v2f mls[4];
  float m = -INFINITY;
#pragma unroll
  for (int s = 0; s < 4; s++) {
    mls[s] = ml[s * 32 + row];
    m = fmaxf(m, mls[s][0]);
  }
  float l = 0.f, wgt[4];
#pragma unroll
  for (int s = 0; s < 4; s++) {
    wgt[s] = __builtin_amdgcn_exp2f(mls[s][0] - m);          // 0 for a wave without blocks (the first wave always has one)
    l = __builtin_fmaf(mls[s][1], wgt[s], l);
  }
  const bool whole = args.nsplit == 1;
  const float inv_l = 1.0f / l;
  if (wave < KS) {
#pragma unroll
    for (int aa = 0; aa < 4; aa++) {
      v4f o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < 4; s++) {
        const v4f x = *(const v4f*)(xch + (((s * KS + wave) * 4 + aa) * 64 + ln) * 4);
#pragma unroll
        for (int e = 0; e < 4; e++) o[e] = __builtin_fmaf(x[e], wgt[s], o[e]);
      }
      const int ch = 32 * wave + 8 * aa + 4 * half;
      if (whole) {
        v4us ob;
#pragma unroll
        for (int e = 0; e < 4; e++) ob[e] = float_to_bf16_bits(o[e] * inv_l);
        *(v4us*)(args.O + args.qview.row(bh, row) + ch) = ob;
      } else {
        *(v4f*)(args.part + (((size_t)bh * args.nsplit + split) * 32 + row) * D + ch) = o;
      }
    }
  }
  if (wave == 0 && half == 0) {
    if (whole) args.LSE[(size_t)bh * args.nq + row] = (m + __builtin_amdgcn_logf(l) - kLog2_127) * kLn2;
    else args.part_ml[((size_t)bh * args.nsplit + split) * 32 + row] = v2f{m, l};
  }
}

// Joins the workgroups' partial (O, m, l): one workgroup of 256 threads per (query, head), D / 4 of them to a row of O.
// Bound by latency: every thread has the loads of its rows in flight while the waves find m and l, each for itself.
// (One thread per channel and all the rows in
// turn: 1 head of 8192 keys, 32 partial results, 7 us more for the call; 16 heads of 8192 keys, 32 queries, 9 us.)
template <int D>
__global__ void __launch_bounds__(256) sage_fwd_decode_join_kernel(DecodeArgs args, int nsplit) {
  constexpr int LANES = D / 4, GROUPS = 256 / LANES;
  __shared__ v4f sums[GROUPS][LANES];
  const int q = blockIdx.x, bh = blockIdx.y, t = threadIdx.x, lane = t & 63;
  const int g = t / LANES, c = t % LANES;
  const v2f* ml = args.part_ml + (size_t)bh * nsplit * 32 + q;
  const float* part = args.part + ((size_t)bh * nsplit * 32 + q) * D + 4 * c;
  float m = -INFINITY;
  for (int s = lane; s < nsplit; s += 64) m = fmaxf(m, ml[(size_t)s * 32][0]);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
  float l = 0.f;
  for (int s = lane; s < nsplit; s += 64) {
    const v2f e = ml[(size_t)s * 32];
    l = __builtin_fmaf(e[1], __builtin_amdgcn_exp2f(e[0] - m), l);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) l += __shfl_xor(l, off, 64);
  v4f o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
  for (int s = g; s < nsplit; s += GROUPS) {
    const float w = __builtin_amdgcn_exp2f(ml[(size_t)s * 32][0] - m);
    const v4f x = *(const v4f*)(part + (size_t)s * 32 * D);
#pragma unroll
    for (int e = 0; e < 4; e++) o[e] = __builtin_fmaf(x[e], w, o[e]);
  }
  sums[g][c] = o;
  __syncthreads();
  if (g != 0) return;
#pragma unroll
  for (int k = 1; k < GROUPS; k++) {
    const v4f x = sums[k][c];
#pragma unroll
    for (int e = 0; e < 4; e++) o[e] += x[e];
  }
  const float inv_l = 1.0f / l;
  v4us ob;
#pragma unroll
  for (int e = 0; e < 4; e++) ob[e] = float_to_bf16_bits(o[e] * inv_l);
  *(v4us*)(args.O + args.qview.row(bh, q) + 4 * c) = ob;
  if (t == 0) args.LSE[(size_t)bh * args.nq + q] = (m + __builtin_amdgcn_logf(l) - kLog2_127) * kLn2;
}

}  // namespace sage
