"""The forward on an odd number of 64-row Q blocks: the last workgroup has two waves without queries."""
import pytest
import torch

from paper_2603_02170_amd import binding

pytestmark = pytest.mark.gpu


# one block, three, a partial last block, non-square with the mask; enough heads that the call takes the full machine's form (more than
# 1024 waves of 32 queries), or numerics blocks of 128 keys, which always do
@pytest.mark.parametrize("Nq,Nk,d,causal,q_smooth,bkv", [(64, 64, 128, True, False, 0), (192, 192, 64, True, False, 0), (300, 300, 128, False, False, 0),
                                                         (160, 224, 128, True, False, 0), (577, 577, 128, True, True, 0), (64, 300, 64, False, False, 128),
                                                         (413, 413, 128, True, False, 128), (320, 200, 64, False, True, 128)])
def test_every_row_has_the_bits_of_a_call_on_a_head_alone(Nq, Nk, d, causal, q_smooth, bkv):
    heads = 1024 // (-(-Nq // 32)) + 9
    g = torch.Generator(device="cuda").manual_seed(Nq + Nk)
    Q, K, V = (torch.randn((1, heads, n, d), generator=g, device="cuda").to(torch.bfloat16) for n in (Nq, Nk, Nk))
    kw = dict(causal=causal, q_smooth=q_smooth, Nkv=Nk, bkv=bkv)
    p, p1 = binding.SageParams(1, heads, Nq, d, **kw), binding.SageParams(1, 1, Nq, d, **kw)
    O, L = torch.full_like(Q, float("nan")), torch.full((1, heads, Nq), float("nan"), device="cuda")
    O, L = binding.sagebwd_fwd(Q, K, V, p, None, O, L)
    for h in (0, heads // 2, heads - 1):
        sl = slice(h, h + 1)
        o, l = binding.sagebwd_fwd(*(t[:, sl].contiguous() for t in (Q, K, V)), p1)
        torch.cuda.synchronize()
        assert torch.isfinite(o.float()).all() and torch.equal(O[:, sl], o) and torch.equal(L[:, sl], l), h


# one Q block and three at d = 64 with so many heads that workgroups of two waves serve them, one head fewer and more, a partial block
@pytest.mark.parametrize("heads,N,causal,bkv", [(769, 64, True, 0), (768, 64, True, 0), (800, 33, False, 0), (800, 64, False, 128), (385, 192, True, 0),
                                                (384, 192, True, 0), (400, 150, True, 0), (400, 192, True, 128), (400, 192, False, 0)])
def test_short_heads_have_the_bits_of_a_call_on_a_head_alone(heads, N, causal, bkv):
    g = torch.Generator(device="cuda").manual_seed(heads + N)
    Q, K, V = (torch.randn((1, heads, N, 64), generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    O, L = torch.full_like(Q, float("nan")), torch.full((1, heads, N), float("nan"), device="cuda")
    binding.sagebwd_fwd(Q, K, V, binding.SageParams(1, heads, N, 64, causal=causal, bkv=bkv), None, O, L)
    for h in (0, heads // 2, heads - 1):
        sl = slice(h, h + 1)
        o, l = binding.sagebwd_fwd(*(t[:, sl].contiguous() for t in (Q, K, V)), binding.SageParams(1, 1, N, 64, causal=causal, bkv=bkv))
        torch.cuda.synchronize()
        assert torch.isfinite(o.float()).all() and torch.equal(O[:, sl], o) and torch.equal(L[:, sl], l), h
