"""O in the memory of Q, K or V, and gradients in that of Q, K and O: the bits of the call on separate tensors."""
import pytest
import torch

from paper_2603_02170_amd import binding

pytestmark = pytest.mark.gpu


def _inputs(heads, Nq, Nk, d):
    g = torch.Generator(device="cuda").manual_seed(100 * Nq + Nk)
    return [torch.randn((1, heads, n, d), generator=g, device="cuda").to(torch.bfloat16) for n in (Nq, Nk, Nk, Nq)]


def _in(buffer, first, shape):
    """A tensor of `shape` in `buffer`, from element `first` on."""
    n = torch.Size(shape).numel()
    return buffer.view(-1)[first:first + n].view(shape)


# several Q blocks a head, of one key block and of two (the forward of short heads), a decoding step, and a length of neither
@pytest.mark.parametrize("heads,Nq,Nk,d,causal", [(40, 128, 128, 128, True), (40, 100, 100, 64, False), (30, 300, 64, 128, False), (64, 4, 1300, 64, False),
                                                  (600, 2, 100, 128, False), (6, 320, 320, 128, True)])
@pytest.mark.parametrize("codes", [False, True])
def test_forward(heads, Nq, Nk, d, causal, codes):
    Q, K, V, _ = _inputs(heads, Nq, Nk, d)
    p = binding.SageParams(1, heads, Nq, d, causal=causal, Nkv=Nk)
    ref = binding.alloc_workspace(p, forward_only=not codes)
    O, L = binding.sagebwd_fwd(Q, K, V, p, ref)
    n, m = Q.numel(), K.numel()
    for where in ("Q", "K", "V", "into Q", "end of K"):
        buf = torch.cat([t.reshape(-1) for t in (Q, K, V)] + [torch.zeros(n, dtype=torch.bfloat16, device="cuda")])
        q, k, v = _in(buf, 0, Q.shape), _in(buf, n, K.shape), _in(buf, n + m, V.shape)
        o = _in(buf, {"Q": 0, "K": n, "V": n + m, "into Q": min(d, n // 2), "end of K": n + m - d}[where], Q.shape)
        ws = binding.alloc_workspace(p, forward_only=not codes)
        o, l = binding.sagebwd_fwd(q, k, v, p, ws, o)
        torch.cuda.synchronize()
        # (a decoding step whose O lies in K or V takes another form: its sums run in another order)
        if Nk > 1000 or (Nq <= 32 and heads * -(-Nk // 64) >= 512):
            assert float((o.double() - O.double()).norm()) <= 2 ** -8 * float(O.double().norm()), where
            assert float((l - L).abs().max()) <= 1e-4, where
        else:
            assert torch.equal(o, O) and torch.equal(l, L), where
        if codes:
            for which in (binding.TENSOR_Q, binding.TENSOR_K, binding.TENSOR_V):
                for a, b in zip(binding.sagebwd_export_quantized(p, ws, which), binding.sagebwd_export_quantized(p, ref, which)):
                    assert torch.equal(a, b), (where, which)


# one block and two of either side (the backward of short heads), and a length that it does not take
@pytest.mark.parametrize("heads,Nq,Nk,d,causal", [(40, 128, 128, 128, True), (300, 33, 33, 64, True), (40, 90, 128, 128, False), (40, 128, 50, 64, False), (6, 200, 200, 128, True)])
def test_backward(heads, Nq, Nk, d, causal):
    Q, K, V, dO = _inputs(heads, Nq, Nk, d)
    for share in (False, True):
        p = binding.SageParams(1, heads, Nq, d, causal=causal, Nkv=Nk, share_quantized=share)
        ws = binding.alloc_workspace(p)
        O, L = binding.sagebwd_fwd(Q, K, V, p, ws)
        want = binding.sagebwd_bwd(Q, K, V, O, dO, L, p, ws)
        n, m = Q.numel(), K.numel()
        # Q, K and O one after the other, and gradients over them: each in its own place, and each a row further on
        for first in (0, d):
            buf = torch.cat([t.reshape(-1) for t in (Q, K, O)] + [torch.zeros(max(n, m) + d, dtype=torch.bfloat16, device="cuda")])
            q, k, o = _in(buf, 0, Q.shape), _in(buf, n, K.shape), _in(buf, n + m, O.shape)
            dq, dk, dv = _in(buf, first, Q.shape), _in(buf, n + first, K.shape), _in(buf, n + m + first, V.shape)
            binding.sagebwd_fwd(Q, K, V, p, ws)
            binding.sagebwd_bwd(q, k, V, o, dO, L, p, ws, dq, dk, dv)
            torch.cuda.synchronize()
            for a, b, name in zip((dq, dk, dv), want, ("dQ", "dK", "dV")):
                assert torch.equal(a, b), (share, first, name)
