// C-ABI host side of the SageBwd library: argument validation, workspace layout,
// kernel launches.  See include/sagebwd.h for the contract of every entry point.
#include "sagebwd.h"

#include <hip/hip_runtime.h>
#include <math.h>
#include <string.h>

#include <mutex>
#include <vector>

#include "common.h"
#include "dispatch.h"
#include "prepass_kernels.h"
#include "fwd_kernel.h"
#include "fwd_decode_kernel.h"
#include "fwd_short_kernel.h"
#include "bwd_kernel.h"
#include "bwd_short_kernel.h"
#include "probe_kernels.h"

// Workspace of sagebwd_fwd_static: one array per GPU, held until the process ends.  In host code the
// name `scratch` is only a handle for hipGetSymbolAddress; the device address it returns (per device)
// is what the kernels are given.
static __device__ __align__(256) unsigned char scratch[SAGEBWD_STATIC_SCRATCH_BYTES];

namespace {

using namespace sage;

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};   // device address of `scratch` on each GPU, looked up once

// Device address of this GPU's copy of `scratch` (the current device's), or nullptr on failure.
void* static_scratch_for_current_device() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (g_scratch_ptr[dev] == nullptr) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess) return nullptr;
    g_scratch_ptr[dev] = ptr;
  }
  return g_scratch_ptr[dev];
}

constexpr size_t kDefaultDsBudget = (size_t)8 << 30;   // bytes of INT8 dS scratch the backward holds at once unless told otherwise

inline size_t align_up(size_t x, size_t a = 256) { return (x + a - 1) / a * a; }

// Rows of every workspace tensor: the caller's N rounded up to the 64-row block.  When the two differ
// the kernels run on the rounded shape: the rows that do not exist are zero rows behind a key mask in
// the workspace, are never read from the caller's tensors (loaders clamp) and never stored.
inline int padded_rows(int N) { return (N + 63) / 64 * 64; }

// Numerics block sizes (rows that share one quantisation scale): 64 unless the caller says 128.
inline int block_q(const sagebwd_params& p) { return p.bq > 0 ? p.bq : 64; }
inline int block_kv(const sagebwd_params& p) { return p.bkv > 0 ? p.bkv : 64; }
inline bool big_blocks(const sagebwd_params& p) { return block_q(p) != 64 || block_kv(p) != 64; }

// Keys per head: N_kv, or N when the caller leaves it 0 (square attention).
inline int kv_len(const sagebwd_params& p) { return p.Nkv > 0 ? p.Nkv : p.N; }

// Where the rows of one of the caller's bf16 tensors start, in elements (times `scale`); `rows` = its
// sequence length (N for Q, O, dO, dQ; N_kv for K, V, dK, dV).
inline RowView caller_view(const sagebwd_params& p, size_t scale, int rows) {
  const size_t N = rows, H = p.H, d = p.d;
  RowView v;
  v.H = p.H;
  if (p.layout == SAGEBWD_LAYOUT_BNHD) {
    v.batch_stride = N * H * d * scale; v.head_stride = d * scale; v.row_stride = H * d * scale;
  } else {
    v.batch_stride = H * N * d * scale; v.head_stride = N * d * scale; v.row_stride = d * scale;
  }
  return v;
}
// Bytes of one of the caller's bf16 tensors of `rows` rows.
inline size_t tensor_bytes(const sagebwd_params& p, int rows) { return (size_t)p.B * p.H * rows * p.d * 2; }

// Byte offsets of every buffer inside the caller's workspace.  What the forward needs comes first
// (`fwd_total` bytes), so that a forward-only caller can pass a much smaller buffer.
struct Workspace {
  size_t kpart, muK, muQ, sQ, sK, sV;
  size_t QF, KF, VT;        // forward operands (QF, KF also feed the backward's S recompute)
  size_t bias;              // Q-smoothing: logit bias table [BH, N/64, N]
  size_t Knorm;             // QK-norm with Q-smoothing: the normalised K as dense bf16 [BH, Nk, d] (the bias kernel reads it)
  size_t QT, KT;            // backward operands (TF layouts) that depend on Q and K only
  size_t fwd_total;         // the forward's need (with SAGEBWD_FLAG_SHARE_QUANTIZED it includes QT, KT)
  size_t sdO, delta, nl2, dOT;
  size_t dSq;               // psi(dS) tiles of one head group [heads_per_group, N/64, N/64, 4096]
  size_t sdS;               // their scales [heads_per_group, N/64, ds_pitch]
  int heads_per_group;      // the backward runs in groups of heads that share the dS scratch
  int ds_pitch;             // tiles per Q-block row of the dS scratch
  size_t tmax;              // B_q = 128: (max P, max |dS|) per tile of the even Q blocks, from the backward's first sweep
  size_t total;
  int nchunk, chunk_rows;   // K-mean reduction: chunks per head, rows per chunk
};

Workspace make_layout(const sagebwd_params& p) {
  Workspace w;
  // Nq, Nk: rows of the Q-like and K-like workspace tensors
  const size_t BH = (size_t)p.B * p.H, Nq = padded_rows(p.N), Nk = padded_rows(kv_len(p)), d = p.d;
  const size_t nqblk = Nq / 64, nkblk = Nk / 64;
  const bool qs = (p.smooth & SAGEBWD_SMOOTH_Q) != 0;
  const bool share = (p.flags & SAGEBWD_FLAG_SHARE_QUANTIZED) != 0;
  w.chunk_rows = mean_chunk_rows((int)BH, kv_len(p));
  w.nchunk = (kv_len(p) + w.chunk_rows - 1) / w.chunk_rows;
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off += align_up(bytes); return o; };
  w.kpart = take(BH * w.nchunk * d * sizeof(double));
  w.muK = take(BH * d * 4);
  w.muQ = take(qs ? BH * nqblk * d * 4 : 0);
  w.sQ = take(BH * nqblk * 4);
  w.sK = take(BH * nkblk * 4);
  w.sV = take(BH * nkblk * 4);
  w.QF = take(BH * Nq * d);
  w.KF = take(BH * Nk * d);
  w.VT = take(BH * Nk * d);
  w.bias = take(qs ? BH * nqblk * Nk * 4 : 0);
  w.Knorm = take(qs && (p.flags & SAGEBWD_FLAG_QK_NORM) ? BH * Nk * d * 2 : 0);
  if (!share) w.fwd_total = off;
  w.QT = take(BH * Nq * d);
  w.KT = take(BH * Nk * d);
  if (share) w.fwd_total = off;
  w.sdO = take(BH * nqblk * 4);
  w.delta = take(BH * Nq * 4);
  w.nl2 = take(BH * Nq * 4);
  w.dOT = take(BH * Nq * d);
  // dS scratch: one 4 KiB tile per (Q block, KV block) and head, capped at the budget by processing the
  // heads in groups.
  // Rows of the dS scratch are three tiles longer than they need to be: with a power-of-two row length
  // the workgroups of the dQ kernel, which walk their rows at the same pace, read addresses that differ
  // in the high bits only (measured: 4 % of that kernel).
  w.ds_pitch = (int)nkblk + 3;
  const size_t ds_head = nqblk * (size_t)w.ds_pitch * 4096;   // bytes of dS scratch per head
  const size_t budget = p.scratch_budget != 0 ? (size_t)p.scratch_budget : kDefaultDsBudget;
  size_t hpg = budget / ds_head;
  if (hpg < 1) hpg = 1;
  if (hpg > BH) hpg = BH;
  w.heads_per_group = (int)hpg;
  w.dSq = take(hpg * ds_head);
  w.sdS = take(hpg * nqblk * (size_t)w.ds_pitch * 4);
  w.tmax = take(block_q(p) == 128 ? hpg * nqblk * (size_t)w.ds_pitch * 8 : 0);
  w.total = off;
  return w;
}

int check_params(const sagebwd_params* p) {
  if (p == nullptr) return SAGEBWD_INVALID_ARG;
  if (p->B <= 0 || p->H <= 0 || p->N <= 0 || p->d <= 0) return SAGEBWD_INVALID_ARG;
  if (p->layout != SAGEBWD_LAYOUT_BHND && p->layout != SAGEBWD_LAYOUT_BNHD) return SAGEBWD_INVALID_ARG;
  if ((p->flags & ~(SAGEBWD_FLAG_SHARE_QUANTIZED | SAGEBWD_FLAG_QK_NORM)) != 0 || p->Nkv < 0 || p->reserved != 0)
    return SAGEBWD_INVALID_ARG;
  if (p->flags & SAGEBWD_FLAG_QK_NORM) {
    if (p->qk_gamma_q == nullptr || p->qk_gamma_k == nullptr || !(p->qk_norm_eps >= 0.f) || isinf(p->qk_norm_eps))
      return SAGEBWD_INVALID_ARG;
  } else if (p->qk_gamma_q != nullptr || p->qk_gamma_k != nullptr) {
    return SAGEBWD_INVALID_ARG;
  }
  if (p->bq < 0 || p->bkv < 0) return SAGEBWD_INVALID_ARG;
  if ((p->smooth & ~(SAGEBWD_SMOOTH_K | SAGEBWD_SMOOTH_Q)) != 0) return SAGEBWD_INVALID_ARG;
  if (p->causal != 0 && p->causal != 1) return SAGEBWD_INVALID_ARG;
  if (!(p->sm_scale >= 0.f) || isinf(p->sm_scale)) return SAGEBWD_INVALID_ARG;
  if (p->d != 64 && p->d != 128) return SAGEBWD_UNSUPPORTED_SHAPE;
  if ((p->bq != 0 && p->bq != 64 && p->bq != 128) || (p->bkv != 0 && p->bkv != 64 && p->bkv != 128))
    return SAGEBWD_UNSUPPORTED_SHAPE;
  const int Nk = kv_len(*p);
  if (p->N > (1 << 30) || Nk > (1 << 30)) return SAGEBWD_UNSUPPORTED_SHAPE;
  // under the mask the last query sits on the last key; the kernels keep one diagonal tile per Q block,
  // which needs the two lengths to differ by whole blocks
  if (p->causal && (Nk < p->N || (Nk - p->N) % 64 != 0)) return SAGEBWD_UNSUPPORTED_SHAPE;
  const double elems = (double)p->B * p->H * (double)padded_rows(p->N > Nk ? p->N : Nk) * p->d;
  if (elems >= 1099511627776.0) return SAGEBWD_UNSUPPORTED_SHAPE;
  if ((double)p->B * p->H > 65535.0) return SAGEBWD_UNSUPPORTED_SHAPE;   // grid.y limit
  return SAGEBWD_OK;
}

float logit_scale(const sagebwd_params& p) {
  return p.sm_scale > 0.f ? p.sm_scale : (float)(1.0 / sqrt((double)p.d));
}

// ---- timing -----------------------------------------------------------------
struct TimedSpan {
  hipEvent_t a, b;
};
// Benchmark hook: the only process-wide state of the library, guarded by one mutex.
std::mutex g_timing_mutex;
int g_timing = 0;   // bit k set: bracket kernel k (sagebwd_kernel) with events
std::vector<TimedSpan> g_spans[SAGEBWD_KERNEL_COUNT];
std::vector<TimedSpan> g_pool;

struct ScopedTimer {
  int k;
  hipStream_t st;
  TimedSpan span;
  bool on;
  ScopedTimer(int kernel, hipStream_t s) : k(kernel), st(s), on(false) {
    std::lock_guard<std::mutex> lock(g_timing_mutex);
    on = ((g_timing >> kernel) & 1) != 0;
    if (!on) return;
    if (!g_pool.empty()) {
      span = g_pool.back();
      g_pool.pop_back();
    } else if (hipEventCreate(&span.a) != hipSuccess || hipEventCreate(&span.b) != hipSuccess) {
      on = false;
      return;
    }
    (void)hipEventRecord(span.a, st);
  }
  ~ScopedTimer() {
    if (!on) return;
    (void)hipEventRecord(span.b, st);
    std::lock_guard<std::mutex> lock(g_timing_mutex);
    g_spans[k].push_back(span);
  }
};

#define SAGE_LAUNCH_CHECK()                                   \
  do {                                                        \
    if (hipGetLastError() != hipSuccess) return SAGEBWD_HIP_ERROR; \
  } while (0)

// ---- pre-pass ---------------------------------------------------------------
// K-mean chunk sums (K-smoothing) into the workspace
template <int D>
int launch_kmean(const void* K, const RowView& kview, const sagebwd_params& p, char* ws, const Workspace& w, const QkNorm& norm,
                 bool own_xcd, hipStream_t st) {
  const auto kernel = norm.gamma != nullptr ? kmean_partial_kernel<D, 4> : own_xcd ? kmean_partial_kernel<D, 0, true> : kmean_partial_kernel<D, 0>;
  const int heads = p.B * p.H;
  kernel<<<prepass_grid(w.nchunk, heads, 1, own_xcd), 256, 0, st>>>((const unsigned short*)K, kview, (double*)(ws + w.kpart), kv_len(p), w.nchunk,
                                                                   w.chunk_rows, norm, heads);
  SAGE_LAUNCH_CHECK();
  return SAGEBWD_OK;
}

template <int D, int SUB>
auto quantiser(int mean) {
  return mean == kMeanOfChunks ? prepass_quant_kernel<D, SUB, kMeanOfChunks> : mean == kMeanInline ? prepass_quant_kernel<D, SUB, kMeanInline>
       : mean == kMeanInlineNormed ? prepass_quant_kernel<D, SUB, kMeanInlineNormed> : prepass_quant_kernel<D, SUB, kMeanInlineNormedBlock>;
}

// want_qk: smooth and quantise Q and K (F layouts; with want_tf also the backward's TF layouts);
// want_v: quantise V; dO != nullptr: quantise dO and form delta and -L*log2(e).
template <int D>
int run_prepass(const void* Q, const void* K, const void* V, const void* dO, const void* O, const float* LSE,
                const sagebwd_params& p, char* ws, const Workspace& w, bool want_qk, bool want_tf, bool want_v,
                hipStream_t st) {
  const int BH = p.B * p.H, Nq = p.N, Nk = kv_len(p), Nqp = padded_rows(Nq), Nkp = padded_rows(Nk);
  const bool ks = (p.smooth & SAGEBWD_SMOOTH_K) != 0;
  const bool qs = (p.smooth & SAGEBWD_SMOOTH_Q) != 0;
  const RowView qview = caller_view(p, 1, Nq), kview = caller_view(p, 1, Nk);     // in bf16 elements
  float* muK = (float*)(ws + w.muK);
  const bool qkn = (p.flags & SAGEBWD_FLAG_QK_NORM) != 0;
  const bool inline_mean = ks && mean_inline(BH, Nk, D);
  const QkNorm norm_q{qkn ? p.qk_gamma_q : nullptr, p.qk_norm_eps}, norm_k{qkn ? p.qk_gamma_k : nullptr, p.qk_norm_eps};
  const int nblk_max = (Nqp > Nkp ? Nqp : Nkp) / 64;
  const bool own_xcd = (want_qk ? ks && !qkn && !qs && prepass_rows_shared(Nqp / 64, Nkp / 64) : dO_own_xcd((long long)BH * Nqp * D)) && !big_blocks(p) && prepass_own_xcd(BH, nblk_max);
  if (want_qk) {
    if (ks && !inline_mean) {
      const int rc = launch_kmean<D>(K, kview, p, ws, w, norm_k, own_xcd, st);
      if (rc != SAGEBWD_OK) return rc;
    }
  }
  QuantJobs jobs;
  memset(&jobs, 0, sizeof(jobs));
  int nj = 0;
  auto q_like = [&](QuantJob& j) { j.view = qview; j.N = Nq; j.Np = Nqp; j.q_like = 1; };
  auto k_like = [&](QuantJob& j) { j.view = kview; j.N = Nk; j.Np = Nkp; j.q_like = 0; };
  if (want_qk) {
    // K first: the mean reduction has just read it, so these blocks find it in the memory-side cache.
    // F layout, and TF layout for the backward (dQ = dS^ K^)
    k_like(jobs.job[nj]);
    jobs.job[nj].src = (const unsigned short*)K;
    jobs.job[nj].outF = (int8_t*)(ws + w.KF);
    jobs.job[nj].outTF = want_tf ? (int8_t*)(ws + w.KT) : nullptr;
    jobs.job[nj].scale = (float*)(ws + w.sK);
    jobs.job[nj].mean_part = ks && !inline_mean ? (const double*)(ws + w.kpart) : nullptr;
    jobs.job[nj].mean_inline = inline_mean;
    jobs.job[nj].nchunk = w.nchunk;
    jobs.job[nj].mu_head_out = muK;
    jobs.job[nj].norm = norm_k;
    jobs.job[nj].norm_out = (qkn && qs) ? (unsigned short*)(ws + w.Knorm) : nullptr;
    nj++;
    // Q: F layout (S = Q^ K^^T in both passes) and, for the backward, TF layout (dK = dS^^T Q^)
    q_like(jobs.job[nj]);
    jobs.job[nj].src = (const unsigned short*)Q;
    jobs.job[nj].outF = (int8_t*)(ws + w.QF);
    jobs.job[nj].outTF = want_tf ? (int8_t*)(ws + w.QT) : nullptr;
    jobs.job[nj].scale = (float*)(ws + w.sQ);
    jobs.job[nj].mu_block_out = qs ? (float*)(ws + w.muQ) : nullptr;
    jobs.job[nj].norm = norm_q;
    nj++;
  }
  if (want_v) {
    // V: TF layout (O = P^ V^ contracts over keys); the backward uses the bf16 V only
    k_like(jobs.job[nj]);
    jobs.job[nj].src = (const unsigned short*)V;
    jobs.job[nj].outTF = (int8_t*)(ws + w.VT);
    jobs.job[nj].scale = (float*)(ws + w.sV);
    nj++;
  }
  if (dO != nullptr) {
    // dO: TF layout (dV = P^^T dO^ contracts over queries), plus delta when O is given
    q_like(jobs.job[nj]);
    jobs.job[nj].src = (const unsigned short*)dO;
    jobs.job[nj].outTF = (int8_t*)(ws + w.dOT);
    jobs.job[nj].scale = (float*)(ws + w.sdO);
    jobs.job[nj].O = (const unsigned short*)O;
    jobs.job[nj].delta = (float*)(ws + w.delta);
    jobs.job[nj].lse = LSE;
    jobs.job[nj].nl2 = (float*)(ws + w.nl2);
    nj++;
  }
  if (nj > 0) {
    // one launch per numerics block size in use (64-row blocks per numerics block: 1 or 2); Q-like jobs
    // quantise per B_q rows, K-like jobs per B_kv rows
    for (int sub = 1; sub <= 2; sub++) {
      QuantJobs part;
      memset(&part, 0, sizeof(part));
      int np = 0;
      for (int k = 0; k < nj; k++) {
        if ((jobs.job[k].q_like ? block_q(p) : block_kv(p)) / 64 == sub) part.job[np++] = jobs.job[k];
      }
      if (np == 0) continue;
      const int blocks = (nblk_max + sub - 1) / sub;
      const dim3 grid = prepass_grid(blocks, BH, np, own_xcd);
      // (numerics blocks of 128 rows: fours unless a head has one block)
      const bool fours = sub == 1 ? normed_rows_by_fours((long long)BH * nblk_max, Nkp / kBlock) : Nk > kBlock;
      const int mean = !(want_qk && inline_mean) ? kMeanOfChunks : !qkn ? kMeanInline : fours ? kMeanInlineNormed : kMeanInlineNormedBlock;
      if (own_xcd) {                    // (numerics blocks of 64, no QK-norm)
        OwnXcdJobs own;
        own.blocks = blocks;
        own.heads = BH;
        memcpy(own.job, part.job, sizeof(own.job));
        const auto kernel = mean == kMeanInline ? prepass_quant_kernel<D, 1, kMeanInline, true> : prepass_quant_kernel<D, 1, kMeanOfChunks, true>;
        kernel<<<grid, 256, 0, st>>>(own);
      } else {
        const auto kernel = sub == 1 ? quantiser<D, 1>(mean) : quantiser<D, 2>(mean);
        kernel<<<grid, 256, 0, st>>>(part);
      }
      SAGE_LAUNCH_CHECK();
    }
  }
  if (qs && want_qk) {
    const float sl2 = logit_scale(p) * 1.4426950408889634f;
    // with QK-norm the bias is formed from the normalised keys, which the quantiser's K blocks left in the workspace
    RowView dense;
    dense.H = p.H;
    dense.batch_stride = (size_t)p.H * Nkp * D; dense.head_stride = (size_t)Nkp * D; dense.row_stride = D;
    const unsigned short* keys = qkn ? (const unsigned short*)(ws + w.Knorm) : (const unsigned short*)K;
    const RowView kv = qkn ? dense : kview;
    const float* muQ = (const float*)(ws + w.muQ);
    float* bias = (float*)(ws + w.bias);
    const int shift = p.causal ? (Nk - Nq) / 64 : -1;
    const dim3 bgrid(Nkp / 64, BH);
    const auto table = use_bias_short(BH, Nkp / 64, Nqp / 64, D) ? qsmooth_bias_short_kernel<D> : qsmooth_bias_kernel<D>;
    table<<<bgrid, 256, 0, st>>>(keys, kv, muK, muQ, bias, Nk, Nkp, Nqp / 64, shift, sl2);
    SAGE_LAUNCH_CHECK();
  }
  return SAGEBWD_OK;
}

template <int D>
int prepass_for_forward(const void* Q, const void* K, const void* V, const sagebwd_params& p, char* ws,
                        const Workspace& w, hipStream_t st) {
  const bool share = (p.flags & SAGEBWD_FLAG_SHARE_QUANTIZED) != 0;
  return run_prepass<D>(Q, K, V, nullptr, nullptr, nullptr, p, ws, w, true, share, true, st);
}
template <int D>
int prepass_for_backward(const void* Q, const void* K, const void* V, const void* dO, const void* O, const float* LSE,
                         const sagebwd_params& p, char* ws, const Workspace& w, bool reuse, hipStream_t st) {
  return run_prepass<D>(Q, K, V, dO, O, LSE, p, ws, w, !reuse, true, false, st);
}

constexpr int kSimds = 4 * kCus;

// Few queries against many keys: split the keys inside the workgroup (sage_fwd_split_kernel) where there are a few tiles
// for each split, while there is a CU for each 64-query workgroup (its LDS takes a whole one), and for two rounds of
// them where the chains are long and several workgroups share a head's keys.  Whole calls, d = 128, us with one chain
// per query -> split: 256 workgroups: 512 x 1024 29.1 -> 25.7, 512 x 4096 82.7 -> 66.9, 128 x 8192 299 -> 285, 64 x 1024
// 67.6 -> 67.2; 320 to 512: 512 x 1024 35.2 -> 38.5, 512 x 2048 58.2 -> 59.2, 128 x 8192 442 -> 461, 512 x 4096 119 -> 116,
// 512 x 8192 235 -> 228; 768: 512 x 4096 170 -> 175.
bool use_fwd_split(const FwdArgs& a) {
  const long long wgs = (long long)a.BH * (a.Nq / 64);
  return a.N >= 2 * a.Nq && a.N >= 8 * kBlock && (wgs <= kCus || (wgs <= 2 * kCus && a.N >= 64 * kBlock && a.Nq >= 8 * kBlock));
}
// At most one wave of sage_fwd_kernel (32 queries) per SIMD: two waves share them (sage_fwd_pair_kernel; same
// bits).  Whole calls at d = 128, us: with the mask N = 1024, 256 waves 30.2 -> 26.0, 1024 waves 35.2 -> 31.2, 1280 42.1 ->
// 40.1, 3072 61.8 -> 66.5; N = 4096, 1024 waves 84.1 -> 67.7, 1280 88.0 -> 84.1; without it N = 1024, 1024 waves 35.7 -> 35.3,
// 1280 42.2 -> 49.1; at d = 64, N = 4096, 1024 waves 67.2 -> 51.3, 1280 69.9 -> 77.2.
bool use_fwd_pair(const FwdArgs& a) { return (long long)a.BH * ((a.Nq + 31) / 32) <= kSimds; }

// Four waves share them (sage_fwd_quad_kernel; same bits).  (A head's codes are addressed with 32 bits.)
bool use_fwd_quad(const FwdArgs& a, int d, bool causal) {
  return (long long)a.N * d <= (1ll << 30) && fwd_quad_is_faster(a.BH, a.N / kBlock, a.Nq / kBlock, d, causal);
}

// the forms for calls that do not fill the machine: 64 queries per workgroup
enum class FwdForm { pair, quad, split };
template <int D, bool CAUSAL, bool QS>
int launch_fwd_small(const FwdArgs& a, FwdForm form, hipStream_t st) {
  FwdArgs args = a;
  args.n_qtiles = a.Nq / 64;
  const int grid = grid_for(a.BH, args.n_qtiles);
  // (the pair form's workgroups share a CU; the other two have one to themselves, the quad form's in up to three rounds under the mask)
  const bool fold = CAUSAL && form == FwdForm::pair && fwd_pair_is_folded(a.BH, a.N / kBlock, a.Nq / kBlock, D);
  const LaunchOrder order = folded_order(a.BH, args.n_qtiles, 2, fold ? 2 : 1);
  args.fold_end = order.fold_end;
  args.head_set = CAUSAL && form == FwdForm::quad ? quad_head_set(a.BH, args.n_qtiles) : order.head_set;
  if (form == FwdForm::quad) sage_fwd_quad_kernel<D, CAUSAL, QS><<<grid, 512, 0, st>>>(args);
  else if (form == FwdForm::split) sage_fwd_split_kernel<D, CAUSAL, QS, 2, 4><<<grid, 512, 0, st>>>(args);
  else sage_fwd_pair_kernel<D, CAUSAL, QS, 2><<<grid, 256, 0, st>>>(args);
  SAGE_LAUNCH_CHECK();
  return SAGEBWD_OK;
}

// One Q block, or three under the mask: half or a quarter of the waves of such workgroups would have no queries.  Workgroups of two waves
// then, at d = 64 (five fit a CU beside their rings, three of four waves; at d = 128 two of either) and once they are more than one round.
// Whole calls, us, four waves -> two: 800 heads of N = 64 18.3 -> 16.1, 1100 22.7 -> 23.1, 1600 30.6 -> 28.8, 4096 60.4 -> 57.1; 300
// heads of N = 192 with the mask 22.7 -> 22.0, 350 24.8 -> 25.3, 400 29.2 -> 27.3, 2048 90.0 -> 85.5; blocks of 128 keys 4096 of 64
// 66.5 -> 63.1, 2048 of 192 94.6 -> 91.6.  Not with five blocks (1000 of N = 320 76.2 -> 78.4), more keys (2048 of 64 x 256 80.6 ->
// 81.3, 1300 55.3 -> 57.3) or Q-smoothing (2048 of 64 48.5 -> 50.0).
bool use_fwd_two_waves(const FwdArgs& a, bool causal) {
  return a.N == a.Nq && (a.Nq == 64 || (causal && a.Nq == 192)) && (long long)a.BH * ((a.Nq + 127) / 128) > 3 * kCus;
}

// Full machines: workgroups of four waves (32 queries each), two (d = 128) or three (d = 64) per CU: the waves that share a SIMD
// then belong to different workgroups and do not wait at each other's barriers (measured 7 % faster than one 8-wave workgroup per
// CU, although that stages every K^/V^ tile once for twice as many queries).  kv128: numerics blocks of 128 keys (the per-token
// quantiser of P~ takes its row max over two tiles).
template <int D, bool CAUSAL, bool QS, int NW>
int launch_fwd_full(const FwdArgs& a, bool kv128, hipStream_t st) {
  FwdArgs args = a;
  args.n_qtiles = (a.Nq + 32 * NW - 1) / (32 * NW);
  const int grid = grid_for(a.BH, args.n_qtiles);
  const bool fold = CAUSAL && (NW == 2 || fwd_is_folded(a.BH, args.n_qtiles, a.Nq / kBlock));
  const LaunchOrder order = folded_order(a.BH, args.n_qtiles, 2, fold ? fwd_per_cu(D) : 1);
  args.head_set = order.head_set;
  args.fold_end = order.fold_end;
  if (kv128) sage_fwd_kernel<D, CAUSAL, QS, NW, true><<<grid, 64 * NW, 0, st>>>(args);
  else sage_fwd_kernel<D, CAUSAL, QS, NW><<<grid, 64 * NW, 0, st>>>(args);
  SAGE_LAUNCH_CHECK();
  return SAGEBWD_OK;
}
template <int D, bool CAUSAL, bool QS>
int launch_fwd_form(const FwdArgs& a, bool kv128, hipStream_t st) {
  if (!kv128 && use_fwd_split(a)) return launch_fwd_small<D, CAUSAL, QS>(a, FwdForm::split, st);
  if (!kv128 && use_fwd_quad(a, D, CAUSAL)) return launch_fwd_small<D, CAUSAL, QS>(a, FwdForm::quad, st);
  if (!kv128 && use_fwd_pair(a)) return launch_fwd_small<D, CAUSAL, QS>(a, FwdForm::pair, st);
  if constexpr (D == 64 && !QS) {
    if (use_fwd_two_waves(a, CAUSAL)) return launch_fwd_full<D, CAUSAL, QS, 2>(a, kv128, st);
  }
  return launch_fwd_full<D, CAUSAL, QS, 4>(a, kv128, st);
}

template <int D>
int launch_fwd(const FwdArgs& a, bool causal, bool qs, bool kv128, hipStream_t st) {
  if (causal) return qs ? launch_fwd_form<D, true, true>(a, kv128, st) : launch_fwd_form<D, true, false>(a, kv128, st);
  return qs ? launch_fwd_form<D, false, true>(a, kv128, st) : launch_fwd_form<D, false, false>(a, kv128, st);
}

template <int D, int MODE, bool KV128 = false>
int launch_bwd(const BwdArgs& a, bool causal, bool qs, hipStream_t st) {
  const int npair = (a.N / 64 + 1) / 2;     // one workgroup per pair of KV blocks
  BwdArgs args = a;
  const int grid = grid_for(a.BH, npair);
  const LaunchOrder order = folded_order(a.BH, npair, 2, causal && MODE == kBwdMaxOnly ? kMaxSweepPerCu : 1);
  args.head_set = order.head_set;
  args.fold_end = order.fold_end;
  if (causal) {
    if (qs) sage_bwd_kernel<D, true, true, MODE, KV128><<<grid, 512, 0, st>>>(args);
    else sage_bwd_kernel<D, true, false, MODE, KV128><<<grid, 512, 0, st>>>(args);
  } else {
    if (qs) sage_bwd_kernel<D, false, true, MODE, KV128><<<grid, 512, 0, st>>>(args);
    else sage_bwd_kernel<D, false, false, MODE, KV128><<<grid, 512, 0, st>>>(args);
  }
  SAGE_LAUNCH_CHECK();
  return SAGEBWD_OK;
}

// One KV block per workgroup (sage_bwd_single_kernel; same bits): while its workgroups are given out in one round, or in two
// where the second is much the lighter (square calls with the mask, walks long enough for that to outweigh what every
// workgroup pays for filling its pipeline); at d = 64, where two of its workgroups share a CU (not with Q-smoothing, which
// needs more registers), at every size but the causal walks of one or two Q blocks.  Whole backward calls, us with two KV
// blocks per workgroup -> with one.  d = 128 with the mask: N = 1024, 256 blocks 60.7 -> 47.1, 512 63.3 -> 57.5, 576 64.8 ->
// 68.7; N = 4096, 512 blocks 182 -> 141, 640 186 -> 198; 510 blocks of N = 640 50.3 -> 50.7, 380 47.8 -> 44.0; 504 of N = 576
// 46.9 -> 51.3; N = 256, 256 blocks 30.4 -> 26.3, 384 33.0 -> 35.4; 64 x 1024, 384 blocks 32.0 -> 37.3; 512 x 4096 79.5 -> 85.0.
// Without: N = 1024, 256 blocks 60.1 -> 49.5, 320 61.2 -> 71.7.  d = 64 with Q-smoothing and the mask: 512 blocks of N = 512
// 37.4 -> 33.4, 384 of N = 256 26.5 -> 26.2, 512 27.8 -> 29.3; d = 64: 256 heads of N = 128 21.3 -> 21.9, of N = 192 34.6 -> 31.2.
bool use_bwd_single(const BwdArgs& a, int d, bool causal, bool qs) {
  const long long blocks = (long long)a.BH * (a.N / 64);
  const bool lighter_second = causal && a.N == a.Nq && a.N >= (d == 64 ? 8 : 10) * kBlock;
  if (blocks <= kCus || (lighter_second && blocks <= 2 * kCus)) return true;
  return d == 64 && !qs && !(causal && a.Nq <= 128);
}
template <int D>
int launch_bwd_single(const BwdArgs& a, bool causal, bool qs, hipStream_t st) {
  const int nblk = a.N / 64;
  BwdArgs args = a;
  const int grid = grid_for(a.BH, nblk);
  const LaunchOrder order = folded_order(a.BH, nblk, 4, causal ? bwd_single_per_cu(D, qs) : 1);
  args.head_set = order.head_set;
  args.fold_end = order.fold_end;
  if (causal) {
    if (qs) sage_bwd_single_kernel<D, true, true><<<grid, 512, 0, st>>>(args);
    else sage_bwd_single_kernel<D, true, false><<<grid, 512, 0, st>>>(args);
  } else {
    if (qs) sage_bwd_single_kernel<D, false, true><<<grid, 512, 0, st>>>(args);
    else sage_bwd_single_kernel<D, false, false><<<grid, 512, 0, st>>>(args);
  }
  SAGE_LAUNCH_CHECK();
  return SAGEBWD_OK;
}

// Four KV blocks per workgroup (sage_bwd_wide_kernel; same bits): d = 128 (Q-smoothing with numerics blocks of 64).
bool use_bwd_wide(const BwdArgs& a, int d, bool causal, bool qs, bool big) {
  return d == 128 && !(qs && big) && bwd_wide_is_faster(a.BH, a.N / kBlock, a.Nq / kBlock, a.shift_blocks, causal);
}
template <bool QSMOOTH, int MODE, bool KV128 = false>
int launch_bwd_wide(const BwdArgs& a, bool causal, hipStream_t st) {
  const int nquad = (a.N / 64 + 3) / 4;
  BwdArgs args = a;
  // Sets of heads at every length under the mask: four blocks of a head share what an XCD's L2 serves, so four heads' operands do not
  // crowd it, and the lightest workgroups of several heads end the launch.  Whole backward, us one head at a time -> in sets: 64 heads
  // of N = 6144 1612 -> 1538, of 8192 2661 -> 2616, of 8256 2703 -> 2685, 24 of 10000 1527 -> 1472, 32 of 12288 2949 -> 2872, 16 of
  // 16384 2482 -> 2490, 8 of 32768 6233 -> 6228.  Without the mask the rule of the other kernels (16 of 16384 4794 one at a time,
  // 4820 in sets).
  args.head_set = head_set_for(nquad, a.BH, causal);
  const int grid = grid_for(a.BH, nquad);
  if (causal) sage_bwd_wide_kernel<128, true, QSMOOTH, MODE, KV128><<<grid, 512, 0, st>>>(args);
  else sage_bwd_wide_kernel<128, false, QSMOOTH, MODE, KV128><<<grid, 512, 0, st>>>(args);
  SAGE_LAUNCH_CHECK();
  return SAGEBWD_OK;
}

template <int D>
int launch_bwd_dq_split(const DqArgs& a, bool causal, bool stream, hipStream_t st) {
  const int nqblk = a.Nq / 64;
  DqArgs args = a;
  args.head_set = head_set_for(nqblk, a.BH, true);
  const int grid = grid_for(a.BH, nqblk);
  if (causal) {
    if (stream) sage_bwd_dq_split_kernel<D, true, true><<<grid, 4 * D, 0, st>>>(args);
    else sage_bwd_dq_split_kernel<D, true, false><<<grid, 4 * D, 0, st>>>(args);
  } else {
    if (stream) sage_bwd_dq_split_kernel<D, false, true><<<grid, 4 * D, 0, st>>>(args);
    else sage_bwd_dq_split_kernel<D, false, false><<<grid, 4 * D, 0, st>>>(args);
  }
  SAGE_LAUNCH_CHECK();
  return SAGEBWD_OK;
}
template <int D>
int launch_bwd_dq(const DqArgs& a, bool causal, bool stream, hipStream_t st) {
  if (use_dq_split(a.BH, a.N / 64, a.Nq / 64, causal)) return launch_bwd_dq_split<D>(a, causal, stream, st);
  const int npair = (a.Nq / 64 + 1) / 2;    // one workgroup per pair of Q blocks
  DqArgs args = a;
  args.head_set = head_set_for(npair, a.BH, true);   // memory-bound: gains from head sets at every length
  const int grid = grid_for(a.BH, npair);
  if (causal) {
    if (stream) sage_bwd_dq_kernel<D, true, true><<<grid, 256, 0, st>>>(args);
    else sage_bwd_dq_kernel<D, true, false><<<grid, 256, 0, st>>>(args);
  } else {
    if (stream) sage_bwd_dq_kernel<D, false, true><<<grid, 256, 0, st>>>(args);
    else sage_bwd_dq_kernel<D, false, false><<<grid, 256, 0, st>>>(args);
  }
  SAGE_LAUNCH_CHECK();
  return SAGEBWD_OK;
}

// One query block of at most 32 rows that sees every key, plain options: see fwd_decode_kernel.h.
bool use_decode(const sagebwd_params& p) {
  return decode_long_enough((long long)p.B * p.H, padded_rows(kv_len(p)) / 64, p.d, (p.smooth & SAGEBWD_SMOOTH_K) != 0) && p.N <= 32 && p.causal == 0 &&
         !(p.smooth & SAGEBWD_SMOOTH_Q) && !(p.flags & SAGEBWD_FLAG_QK_NORM) && !big_blocks(p);
}

template <int D>
int decode_impl(const void* Q, const void* K, const void* V, void* O, float* LSE, const sagebwd_params& p, char* ws, const Workspace& w,
                hipStream_t st) {
  const bool ks = (p.smooth & SAGEBWD_SMOOTH_K) != 0;
  const int BH = p.B * p.H;
  DecodeArgs a;
  a.Q = (const unsigned short*)Q;
  a.K = (const unsigned short*)K;
  a.V = (const unsigned short*)V;
  a.qview = caller_view(p, 1, p.N);
  a.kview = caller_view(p, 1, kv_len(p));
  a.mean_part = ks ? (const double*)(ws + w.kpart) : nullptr;
  a.nchunk = w.nchunk;
  a.O = (unsigned short*)O;
  a.LSE = LSE;
  a.nq = p.N;
  a.nk = kv_len(p);
  a.nblk = padded_rows(a.nk) / 64;
  a.scale_log2e = logit_scale(p) * 1.4426950408889634f;
  a.blocks_per_wave = decode_blocks_per_wave(BH, a.nblk, D);
  const int nsplit = (a.nblk + 4 * a.blocks_per_wave - 1) / (4 * a.blocks_per_wave);
  // the workgroups' partial results lie where K^ would: a workgroup has at least four key blocks (4 * 64 * D bytes) unless
  // it is the last of its head, and leaves at most 32 * (4 D + 8)
  a.part_ml = (v2f*)(ws + w.KF);
  a.part = (float*)(ws + w.KF + align_up((size_t)BH * nsplit * 32 * sizeof(v2f)));
  const bool own_xcd = ks && decode_own_xcd((long long)BH * a.nk * D) && prepass_own_xcd(BH, a.nblk);
  a.nsplit = nsplit;
  a.heads = BH;
  const dim3 grid = prepass_grid(nsplit, BH, 1, own_xcd);
  if (ks) {
    ScopedTimer tm(SAGEBWD_KERNEL_PREPASS_FWD, st);
    const int rc = launch_kmean<D>(K, a.kview, p, ws, w, QkNorm{nullptr, 0.f}, own_xcd, st);
    if (rc != SAGEBWD_OK) return rc;
  }
  ScopedTimer tm(SAGEBWD_KERNEL_FWD, st);
  if (own_xcd) sage_fwd_decode_kernel<D, true, true><<<grid, 256, 0, st>>>(a);
  else if (ks) sage_fwd_decode_kernel<D, true><<<grid, 256, 0, st>>>(a);
  else sage_fwd_decode_kernel<D, false><<<grid, 256, 0, st>>>(a);
  SAGE_LAUNCH_CHECK();
  if (nsplit > 1) {
    sage_fwd_decode_join_kernel<D><<<dim3(p.N, BH), 256, 0, st>>>(a, nsplit);
    SAGE_LAUNCH_CHECK();
  }
  return SAGEBWD_OK;
}

// Short heads: see fwd_short_kernel.h.
bool use_fwd_short(const sagebwd_params& p, bool codes) {
  return fwd_short_is_faster((long long)p.B * p.H, padded_rows(kv_len(p)) / 64, padded_rows(p.N) / 64, p.d, codes, p.N, kv_len(p)) &&
         !(p.smooth & SAGEBWD_SMOOTH_Q) && !(p.flags & SAGEBWD_FLAG_QK_NORM) && !big_blocks(p);
}
template <int D>
int fwd_short_impl(const void* Q, const void* K, const void* V, void* O, float* LSE, const sagebwd_params& p, char* ws, size_t ws_bytes,
                   const Workspace& w, hipStream_t st) {
  const bool share = (p.flags & SAGEBWD_FLAG_SHARE_QUANTIZED) != 0;
  const int BH = p.B * p.H;
  ShortArgs a;
  memset(&a, 0, sizeof(a));
  a.Q = (const unsigned short*)Q;
  a.K = (const unsigned short*)K;
  a.V = (const unsigned short*)V;
  a.qview = caller_view(p, 1, p.N);
  a.kview = caller_view(p, 1, kv_len(p));
  a.O = (unsigned short*)O;
  a.LSE = LSE;
  a.nq = p.N;
  a.nk = kv_len(p);
  a.nqblk = padded_rows(a.nq) / 64;
  a.nkblk = padded_rows(a.nk) / 64;
  a.shift = p.causal ? a.nk - a.nq : 0;
  a.heads = BH;
  a.own_xcd = prepass_own_xcd(BH, a.nqblk);
  a.k_smooth = (p.smooth & SAGEBWD_SMOOTH_K) != 0;
  // Few queries that see all keys have the decoding form's logits, however many heads the call has: by the biased path their LSE would be
  // off by 2e-5.  (Forwards, us, biased -> converting: 8 heads of 1 x 64 6.44 -> 6.50, 64 of 1 x 128 8.73 -> 8.75, 512 of 1 x 64 9.36 -> 9.42.)
  a.converting = p.N <= 32 && p.causal == 0;
  a.scale_log2e = logit_scale(p) * 1.4426950408889634f;
  // the quantised tensors are wanted by a backward that shares them and by the inspection hooks, which take the workspace of sagebwd_bwd
  if (share || ws_bytes >= w.total) {
    a.QF = (int8_t*)(ws + w.QF);
    a.KF = (int8_t*)(ws + w.KF);
    a.VT = (int8_t*)(ws + w.VT);
    a.QT = share ? (int8_t*)(ws + w.QT) : nullptr;
    a.KT = share ? (int8_t*)(ws + w.KT) : nullptr;
    a.sQ = (float*)(ws + w.sQ);
    a.sK = (float*)(ws + w.sK);
    a.sV = (float*)(ws + w.sV);
    a.muK = (float*)(ws + w.muK);
  }
  const dim3 grid = prepass_grid(a.nqblk, BH, 1, a.own_xcd != 0);
  ScopedTimer tm(SAGEBWD_KERNEL_FWD, st);
  auto launch = [&](auto kernel) { kernel<<<grid, 512, 0, st>>>(a); };
  if (p.causal) launch(a.nkblk == 1 ? sage_fwd_short_kernel<D, true, 1> : sage_fwd_short_kernel<D, true, 2>);
  else launch(a.nkblk == 1 ? sage_fwd_short_kernel<D, false, 1> : sage_fwd_short_kernel<D, false, 2>);
  SAGE_LAUNCH_CHECK();
  return SAGEBWD_OK;
}

// The forward on a workspace of `ws_bytes` (at least w.fwd_total; arguments already validated).
int forward_impl(const void* Q, const void* K, const void* V, void* O, float* LSE, const sagebwd_params& p,
                 char* ws, size_t ws_bytes, const Workspace& w, hipStream_t st) {
  int rc;
  // outputs in the memory of inputs: the forms that read K and V while they write O are not taken
  const Memory q{Q, tensor_bytes(p, p.N)}, k{K, tensor_bytes(p, kv_len(p))}, v{V, k.bytes}, o{O, q.bytes};
  const bool apart = fwd_outputs_apart(q, k, v, o, Memory{LSE, (size_t)p.B * p.H * p.N * sizeof(float)});
  const bool leaves_codes = ws_bytes >= ((p.flags & SAGEBWD_FLAG_SHARE_QUANTIZED) ? w.fwd_total : w.total);
  if (apart && use_fwd_short(p, leaves_codes)) {
    return p.d == 64 ? fwd_short_impl<64>(Q, K, V, O, LSE, p, ws, ws_bytes, w, st) : fwd_short_impl<128>(Q, K, V, O, LSE, p, ws, ws_bytes, w, st);
  }
  // (a decoding step quantises Q again behind itself where the codes are left)
  if (apart && use_decode(p) && !(leaves_codes && same(o, q))) {
    rc = p.d == 64 ? decode_impl<64>(Q, K, V, O, LSE, p, ws, w, st) : decode_impl<128>(Q, K, V, O, LSE, p, ws, w, st);
    // the quantised tensors themselves are wanted only by a backward that shares them and by the inspection hooks, which
    // take the workspace of sagebwd_bwd
    if (rc != SAGEBWD_OK || !leaves_codes) return rc;
    ScopedTimer tm(SAGEBWD_KERNEL_PREPASS_FWD, st);
    return p.d == 64 ? prepass_for_forward<64>(Q, K, V, p, ws, w, st) : prepass_for_forward<128>(Q, K, V, p, ws, w, st);
  }
  {
    ScopedTimer tm(SAGEBWD_KERNEL_PREPASS_FWD, st);
    rc = p.d == 64 ? prepass_for_forward<64>(Q, K, V, p, ws, w, st) : prepass_for_forward<128>(Q, K, V, p, ws, w, st);
  }
  if (rc != SAGEBWD_OK) return rc;
  FwdArgs a;
  a.QF = (const int8_t*)(ws + w.QF);
  a.KF = (const int8_t*)(ws + w.KF);
  a.VT = (const int8_t*)(ws + w.VT);
  a.sQ = (const float*)(ws + w.sQ);
  a.sK = (const float*)(ws + w.sK);
  a.sV = (const float*)(ws + w.sV);
  const bool qs = (p.smooth & SAGEBWD_SMOOTH_Q) != 0;
  a.bias = qs ? (const float*)(ws + w.bias) : nullptr;
  a.O = (unsigned short*)O;
  a.oview = caller_view(p, 1, p.N);
  a.LSE = LSE;
  a.BH = p.B * p.H;
  a.N = padded_rows(kv_len(p));
  a.nvalid = kv_len(p);
  a.Nq = padded_rows(p.N);
  a.nq_valid = p.N;
  a.shift = p.causal ? kv_len(p) - p.N : 0;
  a.n_qtiles = 0;
  a.scale_log2e = logit_scale(p) * 1.4426950408889634f;
  {
    ScopedTimer tm(SAGEBWD_KERNEL_FWD, st);
    const bool kv128 = block_kv(p) == 128;
    rc = p.d == 64 ? launch_fwd<64>(a, p.causal != 0, qs, kv128, st) : launch_fwd<128>(a, p.causal != 0, qs, kv128, st);
  }
  return rc;
}

// Short heads: see bwd_short_kernel.h.  (All heads in one group: the launch leaves psi(dS) of every head in the scratch.)
bool use_bwd_short(const sagebwd_params& p, const Workspace& w) {
  const bool share = (p.flags & SAGEBWD_FLAG_SHARE_QUANTIZED) != 0;
  return bwd_short_is_faster((long long)p.B * p.H, p.N, kv_len(p), p.d, share) && !(p.smooth & SAGEBWD_SMOOTH_Q) && !big_blocks(p) &&
         (!(p.flags & SAGEBWD_FLAG_QK_NORM) || share) && w.heads_per_group >= p.B * p.H;
}
template <int D>
int bwd_short_impl(const void* Q, const void* K, const void* V, const void* O, const void* dO, const float* LSE, void* dQ, void* dK, void* dV,
                   const sagebwd_params& p, char* ws, const Workspace& w, hipStream_t st) {
  ShortBwdArgs a;
  memset(&a, 0, sizeof(a));
  a.Q = (const unsigned short*)Q;
  a.K = (const unsigned short*)K;
  a.V = (const unsigned short*)V;
  a.O = (const unsigned short*)O;
  a.dO = (const unsigned short*)dO;
  a.nq = p.N;
  a.nk = kv_len(p);
  a.qview = caller_view(p, 1, a.nq);
  a.kview = caller_view(p, 1, a.nk);
  a.LSE = LSE;
  a.dQ = (unsigned short*)dQ;
  a.dK = (unsigned short*)dK;
  a.dV = (unsigned short*)dV;
  a.nqblk = padded_rows(a.nq) / 64;
  a.nkblk = padded_rows(a.nk) / 64;
  a.shift_blocks = p.causal ? (a.nk - a.nq) / 64 : 0;
  a.k_smooth = (p.smooth & SAGEBWD_SMOOTH_K) != 0;
  a.sm_scale = logit_scale(p);
  a.scale_log2e = a.sm_scale * 1.4426950408889634f;
  a.QF = (int8_t*)(ws + w.QF);
  a.QT = (int8_t*)(ws + w.QT);
  a.KF = (int8_t*)(ws + w.KF);
  a.KT = (int8_t*)(ws + w.KT);
  a.dOT = (int8_t*)(ws + w.dOT);
  a.sQ = (float*)(ws + w.sQ);
  a.sK = (float*)(ws + w.sK);
  a.sdO = (float*)(ws + w.sdO);
  a.delta = (float*)(ws + w.delta);
  a.nl2 = (float*)(ws + w.nl2);
  a.muK = (float*)(ws + w.muK);
  a.dSq = (int8_t*)(ws + w.dSq);
  a.ds_pitch = w.ds_pitch;
  a.sdS = (float*)(ws + w.sdS);
  const bool one = a.nqblk == 1 && a.nkblk == 1, share = (p.flags & SAGEBWD_FLAG_SHARE_QUANTIZED) != 0;
  ScopedTimer tm(SAGEBWD_KERNEL_BWD, st);
  auto launch = [&](auto kernel) { kernel<<<p.B * p.H, 512, 0, st>>>(a); };
  auto pick = [&](auto causal) {
    constexpr bool C = decltype(causal)::value;
    if (one) launch(share ? sage_bwd_short_kernel<D, C, 1, true> : sage_bwd_short_kernel<D, C, 1, false>);
    else launch(share ? sage_bwd_short_kernel<D, C, 2, true> : sage_bwd_short_kernel<D, C, 2, false>);
  };
  if (p.causal) pick(std::true_type{});
  else pick(std::false_type{});
  SAGE_LAUNCH_CHECK();
  return SAGEBWD_OK;
}

// Times `reps` launches of `launch` on `st` with one pair of events around them, after one untimed launch;
// waits for them.  Returns the mean milliseconds per launch through *ms.
template <class F>
int time_probe(F launch, int reps, hipStream_t st, double* ms) {
  hipEvent_t a = nullptr, b = nullptr;
  if (hipEventCreate(&a) != hipSuccess) return SAGEBWD_HIP_ERROR;
  if (hipEventCreate(&b) != hipSuccess) {
    (void)hipEventDestroy(a);
    return SAGEBWD_HIP_ERROR;
  }
  int rc = SAGEBWD_OK;
  launch();
  if (hipEventRecord(a, st) != hipSuccess) rc = SAGEBWD_HIP_ERROR;
  for (int r = 0; r < reps && rc == SAGEBWD_OK; r++) launch();
  if (rc == SAGEBWD_OK && hipEventRecord(b, st) != hipSuccess) rc = SAGEBWD_HIP_ERROR;
  if (rc == SAGEBWD_OK && hipEventSynchronize(b) != hipSuccess) rc = SAGEBWD_HIP_ERROR;
  float t = 0.f;
  if (rc == SAGEBWD_OK && hipEventElapsedTime(&t, a, b) != hipSuccess) rc = SAGEBWD_HIP_ERROR;
  if (rc == SAGEBWD_OK && hipGetLastError() != hipSuccess) rc = SAGEBWD_HIP_ERROR;
  (void)hipEventDestroy(a);
  (void)hipEventDestroy(b);
  *ms = (double)t / reps;
  return rc;
}


}  // namespace

extern "C" {

int sagebwd_workspace_bytes(const sagebwd_params* params, size_t* fwd_bytes, size_t* bwd_bytes) {
  int rc = check_params(params);
  if (rc != SAGEBWD_OK) return rc;
  const Workspace w = make_layout(*params);
  if (fwd_bytes != nullptr) *fwd_bytes = w.fwd_total;
  if (bwd_bytes != nullptr) *bwd_bytes = w.total;
  return SAGEBWD_OK;
}

int sagebwd_quantize(const void* Q, const void* K, const void* V, const void* dO, const void* O,
                     const sagebwd_params* params, void* workspace, size_t workspace_bytes,
                     void* stream) {
  int rc = check_params(params);
  if (rc != SAGEBWD_OK) return rc;
  if (Q == nullptr || K == nullptr || V == nullptr || workspace == nullptr) return SAGEBWD_INVALID_ARG;
  if (O != nullptr && dO == nullptr) return SAGEBWD_INVALID_ARG;
  const Workspace w = make_layout(*params);
  if (workspace_bytes < w.total) return SAGEBWD_WORKSPACE_TOO_SMALL;
  hipStream_t st = (hipStream_t)stream;
  char* ws = (char*)workspace;
  // the inspection pre-pass fills every layout: forward operands first, then the backward's
  {
    ScopedTimer tm(SAGEBWD_KERNEL_PREPASS_FWD, st);
    rc = params->d == 64 ? prepass_for_forward<64>(Q, K, V, *params, ws, w, st)
                         : prepass_for_forward<128>(Q, K, V, *params, ws, w, st);
  }
  if (rc != SAGEBWD_OK || dO == nullptr) return rc;
  {
    ScopedTimer tm(SAGEBWD_KERNEL_PREPASS_BWD, st);
    rc = params->d == 64 ? prepass_for_backward<64>(Q, K, V, dO, O, nullptr, *params, ws, w, false, st)
                         : prepass_for_backward<128>(Q, K, V, dO, O, nullptr, *params, ws, w, false, st);
  }
  return rc;
}

int sagebwd_export_quantized(const sagebwd_params* params, const void* workspace,
                             size_t workspace_bytes, int which, int8_t* q_out, float* scale_out,
                             void* stream) {
  int rc = check_params(params);
  if (rc != SAGEBWD_OK) return rc;
  if (workspace == nullptr) return SAGEBWD_INVALID_ARG;
  const Workspace w = make_layout(*params);
  if (workspace_bytes < w.total) return SAGEBWD_WORKSPACE_TOO_SMALL;
  size_t qoff, soff;
  int transposed;
  switch (which) {
    case SAGEBWD_TENSOR_Q: qoff = w.QF; soff = w.sQ; transposed = 0; break;
    case SAGEBWD_TENSOR_K: qoff = w.KF; soff = w.sK; transposed = 0; break;
    case SAGEBWD_TENSOR_V: qoff = w.VT; soff = w.sV; transposed = 1; break;
    case SAGEBWD_TENSOR_DO: qoff = w.dOT; soff = w.sdO; transposed = 1; break;
    default: return SAGEBWD_INVALID_ARG;
  }
  hipStream_t st = (hipStream_t)stream;
  const char* ws = (const char*)workspace;
  const size_t BH = (size_t)params->B * params->H;
  const bool k_like = which == SAGEBWD_TENSOR_K || which == SAGEBWD_TENSOR_V;
  const int Np = padded_rows(k_like ? kv_len(*params) : params->N);
  if (q_out != nullptr) {
    const size_t n_chunks = BH * Np * params->d / 16;
    export_fragments_kernel<<<(unsigned)((n_chunks + 255) / 256), 256, 0, st>>>(
        (const int8_t*)(ws + qoff), q_out, n_chunks, Np, params->d, transposed);
    SAGE_LAUNCH_CHECK();
  }
  if (scale_out != nullptr) {
    const size_t n = BH * (Np / 64);
    copy_f32_kernel<<<(unsigned)((n + 255) / 256), 256, 0, st>>>((const float*)(ws + soff), scale_out, n, 1.0f);
    SAGE_LAUNCH_CHECK();
  }
  return SAGEBWD_OK;
}

int sagebwd_export_stats(const sagebwd_params* params, const void* workspace, size_t workspace_bytes,
                         float* mu_K, float* mu_Q, float* delta, void* stream) {
  int rc = check_params(params);
  if (rc != SAGEBWD_OK) return rc;
  if (workspace == nullptr) return SAGEBWD_INVALID_ARG;
  const Workspace w = make_layout(*params);
  if (workspace_bytes < w.total) return SAGEBWD_WORKSPACE_TOO_SMALL;
  if (mu_Q != nullptr && !(params->smooth & SAGEBWD_SMOOTH_Q)) return SAGEBWD_INVALID_ARG;
  hipStream_t st = (hipStream_t)stream;
  const char* ws = (const char*)workspace;
  const size_t BH = (size_t)params->B * params->H;
  auto copy = [&](size_t off, float* out, size_t n, float sign = 1.0f) {
    unsigned grid = (unsigned)((n + 255) / 256);
    if (grid > 65535u * 16u) grid = 65535u * 16u;
    copy_f32_kernel<<<grid, 256, 0, st>>>((const float*)(ws + off), out, n, sign);
  };
  if (mu_K != nullptr) { copy(w.muK, mu_K, BH * params->d); SAGE_LAUNCH_CHECK(); }
  const size_t Np = padded_rows(params->N);
  if (mu_Q != nullptr) { copy(w.muQ, mu_Q, BH * (Np / 64) * params->d); SAGE_LAUNCH_CHECK(); }
  if (delta != nullptr) { copy(w.delta, delta, BH * Np, -1.0f); SAGE_LAUNCH_CHECK(); }   // the workspace holds -delta
  return SAGEBWD_OK;
}

int sagebwd_export_ds(const sagebwd_params* params, const void* workspace, size_t workspace_bytes, int head,
                      int8_t* ds_out, float* scale_out, void* stream) {
  int rc = check_params(params);
  if (rc != SAGEBWD_OK) return rc;
  if (workspace == nullptr || head < 0 || head >= params->B * params->H) return SAGEBWD_INVALID_ARG;
  const Workspace w = make_layout(*params);
  if (workspace_bytes < w.total) return SAGEBWD_WORKSPACE_TOO_SMALL;
  // the scratch holds the heads of the LAST group the backward processed: only a backward that ran
  // in one group leaves every head behind
  if (w.heads_per_group < params->B * params->H) return SAGEBWD_UNSUPPORTED_SHAPE;
  const int Nkp = padded_rows(kv_len(*params)), nkblk = Nkp / 64, nqblk = padded_rows(params->N) / 64;
  const char* ws = (const char*)workspace;
  const size_t n = (size_t)nqblk * nkblk * 256;
  export_ds_kernel<<<(unsigned)((n + 255) / 256), 256, 0, (hipStream_t)stream>>>(
      (const int8_t*)(ws + w.dSq) + (size_t)head * nqblk * w.ds_pitch * 4096,
      (const float*)(ws + w.sdS) + (size_t)head * nqblk * w.ds_pitch, ds_out, scale_out, nqblk, Nkp, w.ds_pitch,
      params->causal ? (kv_len(*params) - params->N) / 64 : -1);
  SAGE_LAUNCH_CHECK();
  return SAGEBWD_OK;
}

int sagebwd_fwd(const void* Q, const void* K, const void* V, void* O, float* LSE,
                const sagebwd_params* params, void* workspace, size_t workspace_bytes, void* stream) {
  int rc = check_params(params);
  if (rc != SAGEBWD_OK) return rc;
  if (Q == nullptr || K == nullptr || V == nullptr || O == nullptr || LSE == nullptr || workspace == nullptr)
    return SAGEBWD_INVALID_ARG;
  const Workspace w = make_layout(*params);
  if (workspace_bytes < w.fwd_total) return SAGEBWD_WORKSPACE_TOO_SMALL;
  return forward_impl(Q, K, V, O, LSE, *params, (char*)workspace, workspace_bytes, w, (hipStream_t)stream);
}

int sagebwd_fwd_static(const void* Q, const void* K, const void* V, void* O, float* LSE,
                       const sagebwd_params* params, void* stream) {
  int rc = check_params(params);
  if (rc != SAGEBWD_OK) return rc;
  if (Q == nullptr || K == nullptr || V == nullptr || O == nullptr || LSE == nullptr) return SAGEBWD_INVALID_ARG;
  // the backward of such a call would need the caller's workspace anyway: nothing is shared through `scratch`
  if ((params->flags & SAGEBWD_FLAG_SHARE_QUANTIZED) != 0) return SAGEBWD_INVALID_ARG;
  const Workspace w = make_layout(*params);
  if (w.fwd_total > (size_t)SAGEBWD_STATIC_SCRATCH_BYTES) return SAGEBWD_STATIC_SCRATCH_TOO_SMALL;
  char* ws = (char*)static_scratch_for_current_device();
  if (ws == nullptr) return SAGEBWD_HIP_ERROR;
  // every byte of the forward's workspace that a kernel reads is written earlier in the same call
  // (the pre-pass fills all operand rows, the missing ones of a partial block as zero codes), so nothing
  // the previous call left in the array has to be cleared
  return forward_impl(Q, K, V, O, LSE, *params, ws, w.fwd_total, w, (hipStream_t)stream);
}

int sagebwd_bwd(const void* Q, const void* K, const void* V, const void* O, const void* dO,
                const float* LSE, void* dQ, void* dK, void* dV, const sagebwd_params* params,
                void* workspace, size_t workspace_bytes, void* stream) {
  int rc = check_params(params);
  if (rc != SAGEBWD_OK) return rc;
  if (Q == nullptr || K == nullptr || V == nullptr || O == nullptr || dO == nullptr || LSE == nullptr ||
      dQ == nullptr || dK == nullptr || dV == nullptr || workspace == nullptr)
    return SAGEBWD_INVALID_ARG;
  const Workspace w = make_layout(*params);
  if (workspace_bytes < w.total) return SAGEBWD_WORKSPACE_TOO_SMALL;
  hipStream_t st = (hipStream_t)stream;
  char* ws = (char*)workspace;
  const int BH = params->B * params->H, d = params->d;
  const int Nk = kv_len(*params), Nkp = padded_rows(Nk), Nqp = padded_rows(params->N);
  const int shift_blocks = params->causal ? (Nk - params->N) / 64 : 0;
  const bool qs = (params->smooth & SAGEBWD_SMOOTH_Q) != 0;
  const Memory mq{Q, tensor_bytes(*params, params->N)}, mk{K, tensor_bytes(*params, Nk)};
  const Memory read[5] = {mq, mk, {V, mk.bytes}, {O, mq.bytes}, {dO, mq.bytes}}, written[3] = {{dQ, mq.bytes}, {dK, mk.bytes}, {dV, mk.bytes}};
  if (use_bwd_short(*params, w) && bwd_outputs_apart(read, Memory{LSE, (size_t)BH * params->N * sizeof(float)}, written))
    return d == 64 ? bwd_short_impl<64>(Q, K, V, O, dO, LSE, dQ, dK, dV, *params, ws, w, st) : bwd_short_impl<128>(Q, K, V, O, dO, LSE, dQ, dK, dV, *params, ws, w, st);
  {
    ScopedTimer tm(SAGEBWD_KERNEL_PREPASS_BWD, st);
    const bool reuse = (params->flags & SAGEBWD_FLAG_SHARE_QUANTIZED) != 0;   // Q^, K^ as the forward left them
    rc = d == 64 ? prepass_for_backward<64>(Q, K, V, dO, O, LSE, *params, ws, w, reuse, st)
                 : prepass_for_backward<128>(Q, K, V, dO, O, LSE, *params, ws, w, reuse, st);
    if (rc != SAGEBWD_OK) return rc;
  }
  BwdArgs a;
  a.QF = (const int8_t*)(ws + w.QF);
  a.QT = (const int8_t*)(ws + w.QT);
  a.KF = (const int8_t*)(ws + w.KF);
  a.dOT = (const int8_t*)(ws + w.dOT);
  a.cv = caller_view(*params, 1, Nk);           // in bf16 elements
  a.cvq = caller_view(*params, 1, params->N);
  a.V = (const unsigned short*)V;
  a.dO = (const unsigned short*)dO;
  a.sQ = (const float*)(ws + w.sQ);
  a.sK = (const float*)(ws + w.sK);
  a.sdO = (const float*)(ws + w.sdO);
  a.nL2 = (const float*)(ws + w.nl2);
  a.delta = (const float*)(ws + w.delta);
  a.bias = qs ? (const float*)(ws + w.bias) : nullptr;
  a.muQ = qs ? (const float*)(ws + w.muQ) : nullptr;
  a.dSq = (int8_t*)(ws + w.dSq);
  a.ds_pitch = w.ds_pitch;
  a.sdS = (float*)(ws + w.sdS);
  a.tmax = nullptr;
  const bool big = big_blocks(*params);
  a.dK = (unsigned short*)dK;
  a.dV = (unsigned short*)dV;
  a.N = Nkp;
  a.nvalid = Nk;
  a.Nq = Nqp;
  a.nq_valid = params->N;
  a.shift_blocks = shift_blocks;
  a.sm_scale = logit_scale(*params);
  a.scale_log2e = a.sm_scale * 1.4426950408889634f;
  DqArgs q;
  q.cv = a.cvq;
  q.dSq = a.dSq;
  q.ds_pitch = w.ds_pitch;
  q.sdS = a.sdS;
  q.KT = (const int8_t*)(ws + w.KT);
  q.sK = a.sK;
  q.dQ = (unsigned short*)dQ;
  q.nvalid = params->N;
  q.N = Nkp;
  q.Nq = Nqp;
  q.shift_blocks = shift_blocks;
  q.sm_scale = a.sm_scale * kDqWeight;
  const bool wide_form = d == 128 && !(qs && big);
  for (int h0 = 0, nh = 0; h0 < BH; h0 += nh) {
    nh = bwd_heads_of_group(w.heads_per_group, BH - h0, Nkp / 64, Nqp / 64, shift_blocks, params->causal != 0, wide_form);
    a.bh0 = q.bh0 = h0;
    a.BH = q.BH = nh;
    const DsTraffic ds = ds_traffic(nh, Nkp / 64, Nqp / 64, shift_blocks, d, params->causal != 0);
    const bool causal = params->causal != 0, wide = use_bwd_wide(a, d, causal, qs, big);
    a.stream_ds = ds.store_past;
    q.last_first = ds.load_past && !(wide && ds.store_past);
    {
      ScopedTimer tm(SAGEBWD_KERNEL_BWD, st);
      if (!big && wide) {
        rc = qs ? launch_bwd_wide<true, kBwdFused>(a, causal, st) : launch_bwd_wide<false, kBwdFused>(a, causal, st);
        if (rc != SAGEBWD_OK) return rc;
      } else if (!big && use_bwd_single(a, d, causal, qs)) {
        rc = d == 64 ? launch_bwd_single<64>(a, causal, qs, st) : launch_bwd_single<128>(a, causal, qs, st);
        if (rc != SAGEBWD_OK) return rc;
      } else if (!big) {
        rc = d == 64 ? launch_bwd<64, kBwdFused>(a, causal, qs, st) : launch_bwd<128, kBwdFused>(a, causal, qs, st);
        if (rc != SAGEBWD_OK) return rc;
      } else if (block_q(*params) == 64) {
        // 64 x 128: the numerics block is the pair of tiles a workgroup holds at once
        rc = wide ? launch_bwd_wide<false, kBwdFused, true>(a, causal, st)
             : d == 64 ? launch_bwd<64, kBwdFused, true>(a, causal, qs, st) : launch_bwd<128, kBwdFused, true>(a, causal, qs, st);
        if (rc != SAGEBWD_OK) return rc;
      } else {
        // 128-row Q blocks: phase A alone on the even Q blocks for their tiles' maxima, then the full kernel,
        // which pairs every Q block with its neighbour (see the modes in bwd_kernel.h)
        a.tmax = (float*)(ws + w.tmax);
        rc = d == 64 ? launch_bwd<64, kBwdMaxOnly>(a, causal, qs, st) : launch_bwd<128, kBwdMaxOnly>(a, causal, qs, st);
        if (rc != SAGEBWD_OK) return rc;
        if (wide)
          rc = block_kv(*params) == 128 ? launch_bwd_wide<false, kBwdPairedRows, true>(a, causal, st) : launch_bwd_wide<false, kBwdPairedRows>(a, causal, st);
        else if (block_kv(*params) == 128)
          rc = d == 64 ? launch_bwd<64, kBwdPairedRows, true>(a, causal, qs, st) : launch_bwd<128, kBwdPairedRows, true>(a, causal, qs, st);
        else
          rc = d == 64 ? launch_bwd<64, kBwdPairedRows>(a, causal, qs, st) : launch_bwd<128, kBwdPairedRows>(a, causal, qs, st);
        if (rc != SAGEBWD_OK) return rc;
      }
    }
    {
      ScopedTimer tm(SAGEBWD_KERNEL_BWD_DQ, st);
      rc = d == 64 ? launch_bwd_dq<64>(q, causal, ds.load_past, st) : launch_bwd_dq<128>(q, causal, ds.load_past, st);
      if (rc != SAGEBWD_OK) return rc;
    }
  }
  return rc;
}

int sagebwd_set_timing(int kernels) {
  if (kernels < 0 || kernels > SAGEBWD_TIMING_ALL) return SAGEBWD_INVALID_ARG;
  std::lock_guard<std::mutex> lock(g_timing_mutex);
  g_timing = kernels;
  return SAGEBWD_OK;
}

int sagebwd_read_timing(int kernel, double* total_ms, int* launches) {
  if (kernel < 0 || kernel >= SAGEBWD_KERNEL_COUNT || total_ms == nullptr || launches == nullptr)
    return SAGEBWD_INVALID_ARG;
  double tot = 0.0;
  int n = 0;
  std::lock_guard<std::mutex> lock(g_timing_mutex);
  for (TimedSpan& s : g_spans[kernel]) {
    if (hipEventSynchronize(s.b) != hipSuccess) return SAGEBWD_HIP_ERROR;
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, s.a, s.b) != hipSuccess) return SAGEBWD_HIP_ERROR;
    tot += ms;
    n++;
    g_pool.push_back(s);
  }
  g_spans[kernel].clear();
  *total_ms = tot;
  *launches = n;
  return SAGEBWD_OK;
}

int sagebwd_probe_mfma(int kind, int iters, int reps, void* sink, void* stream, double* ms, double* ops) {
  if (kind < 0 || kind > (SAGEBWD_PROBE_MFMA_BF16 | SAGEBWD_PROBE_MFMA_ZERO_OPERANDS) || iters < 1 || iters > (1 << 20) || reps < 1 ||
      reps > 1000 || sink == nullptr || ms == nullptr || ops == nullptr)
    return SAGEBWD_INVALID_ARG;
  hipStream_t st = (hipStream_t)stream;
  int cus = 0, dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    return SAGEBWD_HIP_ERROR;
  // two workgroups of four waves per CU = two waves per SIMD, eight rounds of them
  const int grid = cus * 2 * 8;
  const bool bf16 = (kind & SAGEBWD_PROBE_MFMA_BF16) != 0;
  const int mask = (kind & SAGEBWD_PROBE_MFMA_ZERO_OPERANDS) ? 0 : -1;
  auto launch = [&]() {
    if (bf16) probe_mfma_kernel<true><<<grid, 256, 0, st>>>(iters, 0x5A6E, mask, (int*)sink);
    else probe_mfma_kernel<false><<<grid, 256, 0, st>>>(iters, 0x5A6E, mask, (int*)sink);
  };
  *ops = (double)grid * 4.0 * iters * 4.0 * 2.0 * 32 * 32 * (bf16 ? 16 : 32);
  return time_probe(launch, reps, st, ms);
}

int sagebwd_probe_stream(int kind, const void* src, void* dst, size_t bytes, int reps, void* sink, void* stream, double* ms) {
  if ((kind != SAGEBWD_PROBE_STREAM_COPY && kind != SAGEBWD_PROBE_STREAM_READ) || src == nullptr || bytes < 16 || bytes % 16 != 0 ||
      reps < 1 || reps > 1000 || sink == nullptr || ms == nullptr || (kind == SAGEBWD_PROBE_STREAM_COPY && dst == nullptr))
    return SAGEBWD_INVALID_ARG;
  if (((uintptr_t)src | (uintptr_t)dst) % 16 != 0) return SAGEBWD_INVALID_ARG;
  hipStream_t st = (hipStream_t)stream;
  int cus = 0, dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    return SAGEBWD_HIP_ERROR;
  const size_t pieces = bytes / 16;
  size_t want = (pieces + 255) / 256;
  const int grid = (int)(want < (size_t)cus * 8 ? want : (size_t)cus * 8);
  const bool copy = kind == SAGEBWD_PROBE_STREAM_COPY;
  auto launch = [&]() {
    if (copy) probe_stream_kernel<true><<<grid, 256, 0, st>>>((const v4i*)src, (v4i*)dst, pieces, 0x5A6E, (int*)sink);
    else probe_stream_kernel<false><<<grid, 256, 0, st>>>((const v4i*)src, nullptr, pieces, 0x5A6E, (int*)sink);
  };
  return time_probe(launch, reps, st, ms);
}

const char* sagebwd_strerror(int status) {
  switch (status) {
    case SAGEBWD_OK: return "ok";
    case SAGEBWD_INVALID_ARG: return "invalid argument (null pointer, bad flag or size)";
    case SAGEBWD_UNSUPPORTED_SHAPE: return "unsupported shape (need d in {64,128}, numerics blocks of 64 or 128, sizes within the stated limits)";
    case SAGEBWD_WORKSPACE_TOO_SMALL: return "workspace too small (see sagebwd_workspace_bytes)";
    case SAGEBWD_HIP_ERROR: return "HIP runtime error";
    case SAGEBWD_STATIC_SCRATCH_TOO_SMALL:
      return "problem too large for the built-in scratch of sagebwd_fwd_static (use sagebwd_fwd with a workspace)";
    default: return "unknown status";
  }
}

}  // extern "C"
