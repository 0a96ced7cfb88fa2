"""The logit biases of Q-smoothing for at most 16 Q blocks (a kernel of their own) against those of a call with one Q block more."""
import pytest
import torch

from paper_2603_02170_amd import binding

pytestmark = pytest.mark.gpu


# The first rows of two calls with the same keys: Nq of them, in one to 16 Q blocks, and 1088, in 17.  Both tables are FP32 sums of d products of magnitude one at most
# (rms 3 by the logit scale), good to 5e-6, which moves LSE by as much and single codes of P by one: 1 / 127 of a probability in a few per mille of the entries.
@pytest.mark.parametrize("Nq,Nk,d,causal,token_major,qk_norm", [
    (64, 65, 128, False, False, False), (192, 700, 64, False, True, False), (1024, 448, 128, False, False, False), (960, 130, 64, False, False, True),
    (1024, 1024, 128, True, False, False), (960, 960, 64, True, False, False), (512, 512, 128, True, True, True)])
def test_tables_of_few_and_of_more_q_blocks_agree(Nq, Nk, d, causal, token_major, qk_norm):
    more = 1088
    g = torch.Generator(device="cuda").manual_seed(Nq + d)
    rand = lambda n: torch.randn((2, 3, n, d), generator=g, device="cuda")
    shift = torch.linspace(-2, 2, d, device="cuda")
    Q, K, V = rand(more) + shift, rand(more if causal else Nk), rand(more if causal else Nk)
    Q, K, V = (t.to(torch.bfloat16) for t in (Q, K, V))
    gains = [1.0 + 0.25 * torch.randn(d, generator=g, device="cuda") for _ in range(2)] if qk_norm else [None, None]
    got = []
    for n in (Nq, more):
        nk = n if causal else Nk
        # (under the mask no key past a row matters to it, but for K's mean)
        p = binding.SageParams(2, 3, n, d, causal=causal, q_smooth=True, k_smooth=not causal, Nkv=nk, token_major=token_major, qk_gamma_q=gains[0], qk_gamma_k=gains[1])
        q, k, v = ((t.transpose(1, 2) if token_major else t).contiguous() for t in (Q[:, :, :n], K[:, :, :nk], V[:, :, :nk]))
        O, L = binding.sagebwd_fwd(q, k, v, p)
        got.append(((O.transpose(1, 2) if token_major else O)[:, :, :Nq].float(), L[:, :, :Nq]))
    torch.cuda.synchronize()
    (o, l), (O, L) = got
    assert torch.isfinite(O).all() and torch.isfinite(L).all()
    assert (l - L).abs().max() < 1e-4
    assert (o - O).norm() < 2e-3 * O.norm()
    # the biases matter: without them LSE is another one
    assert L.std() > 0.05
