"""Sums of K that float64 does not hold exactly: the one-launch forms of short heads add them in the pre-pass's order."""
import pytest
import torch

from paper_2603_02170_amd import binding

pytestmark = pytest.mark.gpu


def _bits(t):
    return t.contiguous().view(torch.int32 if t.dtype == torch.float32 else torch.int16 if t.dtype == torch.bfloat16 else torch.int8)


# one key block and two, whole and partial, few queries and many; heads whose keys the quantiser sums, and so many that another launch does
@pytest.mark.parametrize("heads,Nq,Nk,d", [(3, 64, 64, 128), (5, 100, 100, 128), (4, 130, 33, 64), (8, 128, 128, 64), (600, 128, 128, 128), (900, 65, 128, 64), (1900, 10, 50, 128), (2, 1, 127, 64)])
def test_means_and_codes(heads, Nq, Nk, d):
    g = torch.Generator(device="cuda").manual_seed(Nq + Nk)
    Q, K, V, dO = (torch.randn((1, heads, n, d), generator=g, device="cuda") for n in (Nq, Nk, Nk, Nq))
    # pairs of rows whose large values cancel, at random places: what is left of the small ones depends on the order of the additions
    order = torch.rand((1, heads, Nk, d), generator=g, device="cuda").argsort(2)
    pairs = Nk // 4
    big = torch.randn((1, heads, pairs, d), generator=g, device="cuda") * 2.0 ** 54
    K.scatter_(2, order[:, :, :pairs], big)
    K.scatter_(2, order[:, :, pairs:2 * pairs], -big)
    Q, K, V, dO = (t.to(torch.bfloat16) for t in (Q, K, V, dO))
    kw = dict(causal=False, Nkv=Nk)
    ps, p = binding.SageParams(1, heads, Nq, d, share_quantized=True, **kw), binding.SageParams(1, heads, Nq, d, **kw)
    ws, ref = binding.alloc_workspace(ps), binding.alloc_workspace(ps)
    O, L = binding.sagebwd_fwd(Q, K, V, ps, ws)
    binding.sagebwd_quantize(Q, K, V, ps, ref)
    assert torch.equal(_bits(binding.sagebwd_export_stats(ps, ws)[0]), _bits(binding.sagebwd_export_stats(ps, ref)[0]))
    for a, b in zip(binding.sagebwd_export_quantized(ps, ws, binding.TENSOR_K), binding.sagebwd_export_quantized(ps, ref, binding.TENSOR_K)):
        assert torch.equal(_bits(a), _bits(b))
    # a backward that sums K itself
    own = binding.alloc_workspace(p)
    binding.sagebwd_bwd(Q, K, V, O, dO, L, p, own)
    torch.cuda.synchronize()
    assert torch.equal(_bits(binding.sagebwd_export_stats(p, own)[0]), _bits(binding.sagebwd_export_stats(ps, ref)[0]))
