"""The backward with one KV block per workgroup gives the bits of the one with two: a head alone, and in a call that fills the machine."""
import pytest
import torch

from paper_2603_02170_amd import binding, synth

pytestmark = pytest.mark.gpu


# one Q block, two (the walk is shorter than the stages), three, a partial last block of either side, the mask on the first
# tile of the walk, Q-smoothing, and calls with more queries than keys and the other way round
@pytest.mark.parametrize("Nq,Nk,d,causal,q_smooth", [(64, 64, 128, True, False), (128, 128, 64, True, False), (150, 150, 128, False, False),
                                                     (192, 448, 128, True, False), (577, 577, 128, True, True), (448, 70, 128, False, True),
                                                     (37, 300, 128, False, False), (128, 128, 64, True, True)])
def test_one_kv_block_per_workgroup_gives_the_same_bits(Nq, Nk, d, causal, q_smooth):
    heads = 512 // (-(-Nk // 64)) + 9
    Q, _, _, dO = synth.gaussian_inputs(Nq, d, sigma_qk=1.5, seed=Nq + Nk, heads=heads)
    _, K, V, _ = synth.gaussian_inputs(Nk, d, sigma_qk=1.5, seed=Nk, heads=heads)
    Q, K, V, dO = (t.cuda() for t in (Q, K, V, dO))
    kw = dict(causal=causal, q_smooth=q_smooth, Nkv=Nk)
    p, p1 = binding.SageParams(1, heads, Nq, d, **kw), binding.SageParams(1, 1, Nq, d, **kw)
    O, L = binding.sagebwd_fwd(Q, K, V, p)
    many = binding.sagebwd_bwd(Q, K, V, O, dO, L, p)
    for h in (0, heads - 1):
        sl = slice(h, h + 1)
        one = binding.sagebwd_bwd(*(t[:, sl].contiguous() for t in (Q, K, V, O, dO)), L[:, sl].contiguous(), p1)
        torch.cuda.synchronize()
        for a, b, name in zip(many, one, ("dQ", "dK", "dV")):
            assert torch.equal(a[:, sl], b), (h, name)
