"""At most 32 queries that see all of one or two key blocks: their logits do not depend on how many heads the call has."""
import pytest
import torch

from paper_2603_02170_amd import binding

pytestmark = pytest.mark.gpu


# one head and more, one query and 32, one key block and two, a partial block, unit-RMS rows (logits of small scales)
@pytest.mark.parametrize("heads,Nq,Nk,d,k_smooth", [(1, 1, 64, 128, True), (8, 32, 128, 64, True), (64, 1, 100, 128, True), (40, 4, 13, 64, False), (512, 1, 64, 128, True)])
def test_lse_and_a_head_alone(heads, Nq, Nk, d, k_smooth):
    g = torch.Generator(device="cuda").manual_seed(Nq + Nk)
    Q, K, V = (torch.randn((1, heads, n, d), generator=g, device="cuda") for n in (Nq, Nk, Nk))
    Q, K = (x * torch.rsqrt(x.square().mean(-1, keepdim=True)) for x in (Q, K))
    Q, K, V = (x.to(torch.bfloat16) for x in (Q, K, V))
    kw = dict(causal=False, k_smooth=k_smooth, Nkv=Nk)
    p = binding.SageParams(1, heads, Nq, d, **kw)
    ws = binding.alloc_workspace(p)
    O, L = binding.sagebwd_fwd(Q, K, V, p, ws)

    def stored(which, n):
        codes, scale = binding.sagebwd_export_quantized(p, ws, which)[:2]
        scale = scale.double().cpu().reshape(heads, -1).repeat_interleave(64, 1)[:, :n, None]
        return codes.double().cpu().reshape(heads, -1, d)[:, :n] * scale

    # FP32 exponents of at most 16 are rounded by 2^-20, their sum, its logarithm and an LSE of at most 8 by less than that together
    # (the biased path rounds an exponent by 2^-15)
    ref = torch.logsumexp(stored(binding.TENSOR_Q, Nq) @ stored(binding.TENSOR_K, Nk).transpose(1, 2) / d ** 0.5, -1)
    assert (L.double().cpu().reshape(heads, Nq) - ref).abs().max() <= 4 * 2.0 ** -20
    # and the same bits in a call of many heads
    many = 1024
    big = [torch.cat([t] * (many // heads + 1), 1)[:, :many].contiguous() for t in (Q, K, V)]
    o, l = binding.sagebwd_fwd(*big, binding.SageParams(1, many, Nq, d, **kw))
    torch.cuda.synchronize()
    assert torch.equal(o[:, :heads], O) and torch.equal(l[:, :heads], L)
