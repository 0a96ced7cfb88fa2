"""torch.autograd plumbing around the two calls of the library (no arithmetic of its own).

`sage_attention(Q, K, V, ...)` runs `sagebwd_fwd` and records what `sagebwd_bwd` needs, so that the
INT8 attention can stand where a model calls its attention (paper Sec. 5: SageBwd replaces the
attention of the training run, forward and backward).  Tensors are bf16 CUDA tensors, [B, H, N, d] or,
with `token_major`, [B, N, H, d]; K and V may have another length than Q.  The autograd node is native
(csrc/torch_host.cpp): the backward runs on the engine's thread without the interpreter.
"""
from __future__ import annotations

from . import binding


def sage_attention(Q, K, V, causal: bool = True, k_smooth: bool = True, q_smooth: bool = False, sm_scale: float = 0.0,
                   token_major: bool = False, share_quantized: bool = False, return_lse: bool = False):
    """O (and the log-sum-exp, in the smoothed frame) of INT8 attention, differentiable in Q, K, V.

    share_quantized: keep the forward's workspace until the backward and let it reuse psi(Q), psi(K)
    (Algorithm 2 takes them as inputs); costs that workspace's memory between the two calls."""
    O, L = binding._host().attention(Q, K, V, causal, k_smooth, q_smooth, sm_scale, token_major, share_quantized)
    return (O, L) if return_lse else O
