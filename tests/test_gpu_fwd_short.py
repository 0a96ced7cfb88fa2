"""Heads of one or two key blocks, whose psi and forward are one launch (sage_fwd_short_kernel): its codes, scales and means against the
pre-pass's, O and LSE against the forms for other calls, and a backward on what it leaves in the workspace."""
import pytest
import torch

from paper_2603_02170_amd import binding

pytestmark = pytest.mark.gpu


def _inputs(heads, Nq, Nk, d, kind, token_major):
    g = torch.Generator(device="cuda").manual_seed(1000 * Nq + Nk)
    Q, K, V, dO = (torch.randn((1, heads, n, d), generator=g, device="cuda") for n in (Nq, Nk, Nk, Nq))
    K += torch.randn((1, heads, 1, d), generator=g, device="cuda") * 3
    if kind == "tiny":              # 127 / max|x| overflows in some blocks
        K *= 1e-38
        V *= 1e-38
    Q, K, V, dO = (t.to(torch.bfloat16) for t in (Q, K, V, dO))
    if kind == "nan":
        K[0, 0, 0, 0], V[0, -1, -1, -1] = float("inf"), float("nan")
    if kind == "zero":
        V[0, 0] = 0
        Q[0, -1] = 0
    if token_major:
        Q, K, V, dO = (t.permute(0, 2, 1, 3).contiguous() for t in (Q, K, V, dO))
    return Q, K, V, dO


def _bits(t):
    return t.contiguous().view(torch.int16 if t.dtype == torch.bfloat16 else torch.int32 if t.dtype == torch.float32 else torch.int8)


# the smallest call, a full block and one row more and less, two blocks, a partial second one, more and fewer queries than keys, the mask
# with a shift, every Q block taking its turn at the codes; heads with an XCD of their own (8) and without
SHAPES = [(1, 1, 1, 64, False), (3, 64, 64, 128, True), (8, 63, 63, 128, True), (8, 65, 65, 64, True), (5, 128, 128, 128, True), (2, 100, 100, 64, False),
          (8, 64, 128, 128, True), (3, 40, 104, 64, True), (2, 33, 128, 128, False), (4, 300, 64, 128, False), (8, 200, 90, 64, False), (1, 128, 1, 128, False)]


@pytest.mark.parametrize("kind", ["plain", "tiny", "nan", "zero"])
@pytest.mark.parametrize("heads,Nq,Nk,d,causal", SHAPES)
def test_codes_and_a_backward_on_them(heads, Nq, Nk, d, causal, kind):
    for k_smooth, token_major in ((True, False), (False, True)):
        Q, K, V, dO = _inputs(heads, Nq, Nk, d, kind, token_major)
        kw = dict(causal=causal, k_smooth=k_smooth, token_major=token_major, Nkv=Nk)
        p, ps = binding.SageParams(1, heads, Nq, d, **kw), binding.SageParams(1, heads, Nq, d, share_quantized=True, **kw)
        ws, ref = binding.alloc_workspace(ps), binding.alloc_workspace(ps)
        ws.fill_(0x5a)
        ref.fill_(0x5a)
        O, L = binding.sagebwd_fwd(Q, K, V, ps, ws)
        binding.sagebwd_quantize(Q, K, V, ps, ref)
        for which in (binding.TENSOR_Q, binding.TENSOR_K, binding.TENSOR_V):
            for a, b in zip(binding.sagebwd_export_quantized(ps, ws, which), binding.sagebwd_export_quantized(ps, ref, which)):
                assert torch.equal(_bits(a), _bits(b)), which
        assert torch.equal(_bits(binding.sagebwd_export_stats(ps, ws)[0]), _bits(binding.sagebwd_export_stats(ps, ref)[0]))
        # on a workspace of the forward alone nothing is kept; a backward that quantises Q and K itself has the same operands
        o, l = binding.sagebwd_fwd(Q, K, V, p, binding.alloc_workspace(p, forward_only=True))
        assert torch.equal(_bits(O), _bits(o)) and torch.equal(_bits(L), _bits(l))
        shared = binding.sagebwd_bwd(Q, K, V, O, dO, L, ps, ws)
        own = binding.sagebwd_bwd(Q, K, V, O, dO, L, p, binding.alloc_workspace(p))
        torch.cuda.synchronize()
        for a, b in zip(shared, own):
            assert torch.equal(_bits(a), _bits(b))


# Rows do not depend on the other Q blocks of a call without the mask: three Q blocks with so many heads that the call takes the forms for
# full machines, against one and two of them, which come here
@pytest.mark.parametrize("heads,Nk,d,k_smooth", [(176, 128, 128, True), (176, 65, 64, True), (171, 100, 128, False), (171, 128, 64, False)])
def test_rows_have_the_bits_of_a_call_with_more_queries(heads, Nk, d, k_smooth):
    g = torch.Generator(device="cuda").manual_seed(Nk)
    Q, K, V = (torch.randn((1, heads, n, d), generator=g, device="cuda").to(torch.bfloat16) for n in (192, Nk, Nk))
    V[0, 0] *= 30
    Q[0, 1] *= 100                   # logits that take the converting path
    O, L = binding.sagebwd_fwd(Q, K, V, binding.SageParams(1, heads, 192, d, causal=False, k_smooth=k_smooth, Nkv=Nk))
    for first, n in ((0, 64), (64, 128)):
        o, l = binding.sagebwd_fwd(Q[:, :, first:first + n].contiguous(), K, V, binding.SageParams(1, heads, n, d, causal=False, k_smooth=k_smooth, Nkv=Nk))
        torch.cuda.synchronize()
        assert torch.equal(O[:, :, first:first + n], o) and torch.equal(L[:, :, first:first + n], l)


# Few queries of many heads, no mask: the decoding form's calls where their heads are longer.  Its LSE is within a few roundings of the
# log-sum-exp of the stored codes: FP32 exponents of at most 16 are rounded by 2^-20 (and by 2^-15 on the biased path, which is not
# taken here), their sum, its logarithm and an LSE of at most 8 by less than that together.
@pytest.mark.parametrize("heads,Nq,Nk,d,k_smooth", [(1368, 4, 13, 128, False), (921, 26, 102, 128, True), (600, 32, 128, 64, True), (549, 1, 65, 128, True)])
def test_lse_of_few_queries_of_many_heads(heads, Nq, Nk, d, k_smooth):
    g = torch.Generator(device="cuda").manual_seed(5)
    Q, K, V = (torch.randn((1, heads, n, d), generator=g, device="cuda") for n in (Nq, Nk, Nk))
    Q, K = (x * torch.rsqrt(x.square().mean(-1, keepdim=True)) for x in (Q, K))
    Q, K, V = (x.to(torch.bfloat16) for x in (Q, K, V))
    p = binding.SageParams(1, heads, Nq, d, causal=False, k_smooth=k_smooth, Nkv=Nk)
    ws = binding.alloc_workspace(p)
    _, L = binding.sagebwd_fwd(Q, K, V, p, ws)

    def stored(which, n):
        codes, scale = binding.sagebwd_export_quantized(p, ws, which)[:2]
        scale = scale.double().cpu().reshape(heads, -1).repeat_interleave(64, 1)[:, :n, None]
        return codes.double().cpu().reshape(heads, -1, d)[:, :n] * scale

    ref = torch.logsumexp(stored(binding.TENSOR_Q, Nq) @ stored(binding.TENSOR_K, Nk).transpose(1, 2) / d ** 0.5, -1)
    assert (L.double().cpu().reshape(heads, Nq) - ref).abs().max() <= 4 * 2.0 ** -20
