"""The logit biases of Q-smoothing for at most 16 Q blocks: the kernel that few heads take gives the bits of the one that many take."""
import pytest
import torch

from paper_2603_02170_amd import binding

pytestmark = pytest.mark.gpu


# The first heads of two calls of the same sizes: of 2, whose key blocks have a CU each, and of so many that there are more than two per CU
# (use_bias_short).  Both tables contract the channels in one order, and the other kernels that the number of heads chooses give the same bits where the keys
# are fewer than twice the queries.  One Q block, whole and partial last blocks, 16 of them, more keys than queries, fewer.
@pytest.mark.parametrize("Nq,Nk,d,causal,token_major,qk_norm", [
    (64, 65, 128, False, False, False), (41, 41, 128, True, False, False), (192, 350, 64, False, True, False), (1024, 448, 128, False, False, False), (960, 130, 64, False, False, True),
    (1024, 1024, 128, True, False, False), (960, 960, 64, True, False, False), (700, 892, 128, True, False, False), (512, 512, 128, True, True, True)])
def test_tables_of_few_and_of_many_heads_agree(Nq, Nk, d, causal, token_major, qk_norm):
    few, many = 2, 2 * 256 // (-(-Nk // 64)) + 2
    g = torch.Generator(device="cuda").manual_seed(Nq + d)
    rand = lambda n: torch.randn((1, many, n, d), generator=g, device="cuda")
    Q, K, V = rand(Nq) + torch.linspace(-2, 2, d, device="cuda"), rand(Nk), rand(Nk)
    gains = [1.0 + 0.25 * torch.randn(d, generator=g, device="cuda") for _ in range(2)] if qk_norm else [None, None]
    got = []
    for heads in (few, many):
        p = binding.SageParams(1, heads, Nq, d, causal=causal, q_smooth=True, Nkv=Nk, token_major=token_major, qk_gamma_q=gains[0], qk_gamma_k=gains[1])
        q, k, v = (t[:, :heads].to(torch.bfloat16) for t in (Q, K, V))
        q, k, v = ((t.transpose(1, 2) if token_major else t).contiguous() for t in (q, k, v))
        O, L = binding.sagebwd_fwd(q, k, v, p)
        got.append(((O.transpose(1, 2) if token_major else O)[:, :few], L[:, :few]))
    torch.cuda.synchronize()
    (o, l), (O, L) = got
    assert torch.isfinite(O.float()).all() and torch.isfinite(L).all()
    assert torch.equal(l, L) and torch.equal(o, O)
    # the biases matter: without them LSE is another one
    assert L.std() > 0.05
