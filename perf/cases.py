"""The work that users of this library have it do, as cases to be timed and compared.

A case names one pass through the public entry points:

  api = "step"      one training step's attention on a kept workspace and kept gradient buffers: `sagebwd_fwd`, then
                    `sagebwd_bwd`, which takes the quantised Q and K from the forward (`share_quantized`)
  api = "autograd"  the same through `sage_attention` and torch.autograd, as a model's module calls it: outputs and
                    workspaces come from torch's allocator on every call, the backward quantises Q and K itself
  api = "fwd"       `sagebwd_fwd` alone on a kept workspace: prefill, evaluation, decoding against a cache
  api = "static"    `sagebwd_fwd_static`: the forward that takes no workspace

and its tensors: B, H, N query rows, Nkv keys, head dimension d, and the options of `SageParams`.  `inputs` is "normed"
(QK-normed N(0, 1), what a model with QK-norm hands over), "outlier" (no QK-norm: channel offsets in K, some amplified
channels in Q) or "small_grad" (normed, with an upstream gradient of variance 1e-2).
"""
from __future__ import annotations

import math

import torch

from paper_2603_02170_amd import binding
from paper_2603_02170_amd.autograd import sage_attention

_DEFAULTS = dict(api="step", B=1, H=1, N=64, Nkv=0, d=128, causal=True, k_smooth=True, q_smooth=False, token_major=False,
                 qk_norm=False, block=64, inputs="normed")


def _case(**kw):
    return {**_DEFAULTS, **kw}


def listed():
    return [
        # The smallest training step (the tiny shape of the repository's workloads) as a model runs it: launches and
        # host work are all there is.
        _case(name="tiny_autograd", api="autograd", B=1, H=2, N=128, d=64),
        # A short prompt of odd length in a serving loop that owns no workspace.
        _case(name="serve_short", api="static", B=1, H=8, N=1000),
        # One decoding step of two sequences against a cache: one query row per head, every key visible.
        _case(name="decode", api="fwd", B=2, H=32, N=1, Nkv=8192, causal=False),
        # Chunked prefill: the newest 512 tokens against a cache of 4096.
        _case(name="chunked_prefill", api="fwd", B=1, H=32, N=512, Nkv=4096),
        # Ragged batch of a small model through autograd: token-major activations, d = 64, 12 heads, odd length.
        _case(name="ragged_autograd", api="autograd", B=3, H=12, N=1777, d=64, token_major=True),
        # The pre-training shape of the repository's workloads.
        _case(name="pretrain", B=4, H=16, N=2048),
        # The same length with the model's QK-norm fused into the pre-pass and numerics blocks of 128.
        _case(name="qknorm_blocks128", B=2, H=16, N=2048, qk_norm=True, block=128),
        # Outlier stress: no QK-norm, so the logits take the converting path.
        _case(name="outlier", B=2, H=16, N=4096, inputs="outlier"),
        # Prefill / evaluation at the headline shape: the forward alone.
        _case(name="headline_fwd", api="fwd", B=2, H=32, N=8192),
        # The headline training step, the same with Q-smoothing, and the long-context one.
        _case(name="headline", B=2, H=32, N=8192),
        _case(name="headline_qsmooth", B=2, H=32, N=8192, q_smooth=True),
        _case(name="long", B=1, H=32, N=32768, causal=False, inputs="small_grad"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: 1 to 256 heads, 33 to 32768 rows (1 to 16 query rows when decoding), odd lengths
    among them, at most a third of the long-context case's operations (some options cost more per operation)."""
    kind = rng.choice(["step", "step", "step", "autograd", "autograd", "fwd", "fwd", "static", "decode", "chunk", "cross"])
    while True:
        c = _case(api={"decode": "fwd", "chunk": "fwd", "cross": "step"}.get(kind, kind))
        c["B"], c["H"] = _log_int(rng, 1, 8), _log_int(rng, 1, 32)
        c["d"] = rng.choice([64, 128, 128])
        n = _log_int(rng, 33, 32768)
        if rng.random() < 0.5:
            n = max(64, n // 64 * 64)
        c["N"], c["causal"] = n, rng.random() < 0.7
        if kind == "decode":
            c["N"], c["Nkv"], c["causal"] = _log_int(rng, 1, 16), n, False
        elif kind == "chunk":
            c["Nkv"], c["causal"] = n + 64 * _log_int(rng, 1, 128), True
        elif kind == "cross":
            c["Nkv"], c["causal"] = _log_int(rng, 33, 8192), False
        c["token_major"] = rng.random() < 0.3
        c["k_smooth"] = rng.random() < 0.9
        c["q_smooth"] = rng.random() < 0.15
        c["inputs"] = rng.choice(["normed", "normed", "normed", "outlier", "small_grad"])
        if c["api"] in ("step", "fwd"):      # options of SageParams that sage_attention does not take
            c["block"] = 128 if rng.random() < 0.15 else 64
            c["qk_norm"] = c["inputs"] != "outlier" and rng.random() < 0.2
        if _pairs(c) * c["d"] * 14 > 2e13:
            continue
        if c["api"] == "static" and _static_bytes(c) > binding.STATIC_SCRATCH_BYTES:
            continue
        return c


def _static_bytes(c):
    """A generous estimate of the forward's workspace: three INT8 tensors, the bias table of Q-smoothing, small vectors."""
    heads, rows = c["B"] * c["H"], c["N"] + 64
    return int(1.1 * heads * rows * (3 * c["d"] + (rows / 16 if c["q_smooth"] else 0))) + (1 << 20)


def _pairs(c):
    """Visible (query, key) pairs over all heads."""
    n, m = c["N"], c["Nkv"] or c["N"]
    per = n * (m - n) + n * (n + 1) // 2 if c["causal"] else n * m
    return c["B"] * c["H"] * per


def _params(c, gains=(None, None)):
    b = 0 if c["block"] == 64 else c["block"]
    return binding.SageParams(c["B"], c["H"], c["N"], c["d"], causal=c["causal"], k_smooth=c["k_smooth"],
                              q_smooth=c["q_smooth"], token_major=c["token_major"], share_quantized=c["api"] == "step",
                              bq=b, bkv=b, Nkv=c["Nkv"], qk_gamma_q=gains[0], qk_gamma_k=gains[1])


def prepare(case, seed):
    c = {**_DEFAULTS, **case}
    g = torch.Generator(device="cuda").manual_seed(seed)
    B, H, d, n, m = c["B"], c["H"], c["d"], c["N"], c["Nkv"] or c["N"]

    def randn(rows, std=1.0):
        return torch.randn((B, H, rows, d), generator=g, device="cuda", dtype=torch.float32).mul_(std)

    def rms_norm(x):
        return x.mul_(torch.rsqrt(x.square().mean(-1, keepdim=True).add_(1e-6)))

    def held(x):     # bf16, in the caller's layout
        x = x.to(torch.bfloat16)
        return x.permute(0, 2, 1, 3).contiguous() if c["token_major"] else x

    def q_like(x):
        if c["inputs"] == "outlier":     # 1 % of the (head, channel) pairs are amplified
            pick = torch.rand((B, H, 1, d), generator=g, device="cuda") < 0.01
            return torch.where(pick, x * 20.0, x)
        return x if c["qk_norm"] else rms_norm(x)

    def k_like(x):
        if c["inputs"] == "outlier":     # an offset per channel, shared by the tokens
            return x.add_(torch.randn((B, H, 1, d), generator=g, device="cuda") * 5.0)
        return x if c["qk_norm"] else rms_norm(x)

    s = {"case": c}
    s["Q"], s["K"], s["V"] = held(q_like(randn(n))), held(k_like(randn(m))), held(randn(m))
    trains = c["api"] in ("step", "autograd")
    if trains:
        s["dO"] = held(randn(n, 0.1 if c["inputs"] == "small_grad" else 1.0))
    if c["api"] == "autograd":
        for k in "QKV":
            s[k].requires_grad_()
        return s
    gains = (None, None)
    if c["qk_norm"]:
        gains = tuple(1.0 + 0.25 * torch.randn(d, generator=g, device="cuda", dtype=torch.float32) for _ in range(2))
    s["p"] = p = _params(c, gains)
    s["O"] = torch.empty_like(s["Q"])
    s["L"] = torch.empty((B, H, n), dtype=torch.float32, device="cuda")
    if c["api"] != "static":
        s["ws"] = binding.alloc_workspace(p, forward_only=not trains)
    if trains:
        s["dQ"], s["dK"], s["dV"] = torch.empty_like(s["Q"]), torch.empty_like(s["K"]), torch.empty_like(s["V"])
    return s


def run(s):
    api = s["case"]["api"]
    if api == "autograd":
        c = s["case"]
        O, L = sage_attention(s["Q"], s["K"], s["V"], causal=c["causal"], k_smooth=c["k_smooth"], q_smooth=c["q_smooth"],
                              token_major=c["token_major"], return_lse=True)
        dQ, dK, dV = torch.autograd.grad(O, (s["Q"], s["K"], s["V"]), s["dO"])
        return {"O": O.detach(), "L": L, "dQ": dQ, "dK": dK, "dV": dV}
    if api == "static":
        O, L = binding.sagebwd_fwd_static(s["Q"], s["K"], s["V"], s["p"], s["O"], s["L"])
        return {"O": O, "L": L}
    O, L = binding.sagebwd_fwd(s["Q"], s["K"], s["V"], s["p"], s["ws"], s["O"], s["L"])
    if api == "fwd":
        return {"O": O, "L": L}
    dQ, dK, dV = binding.sagebwd_bwd(s["Q"], s["K"], s["V"], O, s["dO"], L, s["p"], s["ws"], s["dQ"], s["dK"], s["dV"])
    return {"O": O, "L": L, "dQ": dQ, "dK": dK, "dV": dV}


def work(case):
    """Forward: Q, K, V read, O and L written, two products per visible pair of rows; a step also reads dO, writes dQ, dK, dV
    and takes five more products."""
    c = {**_DEFAULTS, **case}
    trains = c["api"] in ("step", "autograd")
    q = 2 * c["B"] * c["H"] * c["N"] * c["d"]
    k = 2 * c["B"] * c["H"] * (c["Nkv"] or c["N"]) * c["d"]
    nbytes = 2 * q + 2 * k + 4 * c["B"] * c["H"] * c["N"] + (2 * q + 2 * k if trains else 0)
    return {"bytes": nbytes, "flops": (14 if trains else 4) * _pairs(c) * c["d"]}


def tolerance(case):
    """bf16 outputs of INT8 products: the quantisers inside the loops round values that depend on exp2 and on the order of
    FP32 sums, so single codes may fall to the other side of a step."""
    return {"rel": 5e-3, "max": 0.3}
