"""The backward of heads of at most two blocks of queries and of keys, which is one launch (sage_bwd_short_kernel), against the forms for
other calls: a scratch budget of one head makes the same call take those."""
import pytest
import torch

from paper_2603_02170_amd import binding

pytestmark = pytest.mark.gpu


def _bits(t):
    return t.contiguous().view(torch.int16 if t.dtype == torch.bfloat16 else torch.int32 if t.dtype == torch.float32 else torch.int8)


# the smallest call, full blocks and one row more and less, a partial second block, one block of queries against two of keys and the other
# way round, the mask with a shift
@pytest.mark.parametrize("Nq,Nk,causal", [(1, 1, False), (64, 64, True), (63, 63, True), (65, 65, True), (128, 128, True), (100, 100, False), (128, 128, False),
                                          (64, 128, True), (40, 104, True), (33, 128, False), (128, 1, False), (90, 64, False)])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("kind", ["plain", "nan", "zero"])
def test_bits_of_the_forms_for_other_calls(Nq, Nk, causal, d, kind):
    heads = 3
    g = torch.Generator(device="cuda").manual_seed(1000 * Nq + Nk)
    Q, K, V, dO = (torch.randn((1, heads, n, d), generator=g, device="cuda").to(torch.bfloat16) for n in (Nq, Nk, Nk, Nq))
    Q[0, 1] *= 20
    if kind == "nan":
        V[0, 0, 0, 0], dO[0, 2, -1, -1] = float("inf"), float("nan")
    if kind == "zero":
        dO[0, 0] = 0
        V[0, 1] = 0
    gains = [1.0 + 0.25 * torch.randn(d, generator=g, device="cuda") for _ in range(2)]
    for share, k_smooth, token_major, qk_norm in ((True, True, False, False), (False, True, True, False), (False, False, False, False), (True, True, True, True)):
        q, k, v, do = ((t.permute(0, 2, 1, 3).contiguous() if token_major else t) for t in (Q, K, V, dO))
        kw = dict(causal=causal, k_smooth=k_smooth, token_major=token_major, Nkv=Nk, share_quantized=share)
        if qk_norm:
            kw.update(qk_gamma_q=gains[0], qk_gamma_k=gains[1])
        left = []
        for budget in (0, 1):
            p = binding.SageParams(1, heads, Nq, d, scratch_budget=budget, **kw)
            ws = binding.alloc_workspace(p)
            ws.fill_(0x5a)
            O, L = binding.sagebwd_fwd(q, k, v, p, ws)
            if kind == "nan":
                O = torch.nan_to_num(O)
            grads = [torch.full_like(t, 7.0) for t in (q, k, v)]
            binding.sagebwd_bwd(q, k, v, O, do, L, p, ws, *grads)
            mu, _, delta = binding.sagebwd_export_stats(p, ws, want_delta=True)
            codes = [t for which in (binding.TENSOR_Q, binding.TENSOR_K, binding.TENSOR_DO) for t in binding.sagebwd_export_quantized(p, ws, which)]
            left.append(grads + [mu, delta] + codes)
        torch.cuda.synchronize()
        for n, (a, b) in enumerate(zip(*left)):
            assert torch.equal(_bits(a), _bits(b)), (share, k_smooth, token_major, qk_norm, n)
