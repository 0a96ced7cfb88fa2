"""dQ of calls that do not fill the machine (one Q block per workgroup) has the bits of the form with two Q blocks per workgroup."""
import pytest
import torch

from paper_2603_02170_amd import binding

pytestmark = pytest.mark.gpu


# two stages an interval, two intervals ahead: walks of two to nine stages, odd and even, whole and partial last Q blocks, more keys than queries with the
# mask and without; both tensor layouts; numerics blocks of 128
@pytest.mark.parametrize("Nq,Nk,d,causal,token_major,block", [
    (128, 128, 128, True, False, 0), (129, 129, 64, True, False, 0), (192, 192, 128, True, True, 0), (300, 300, 128, True, False, 0), (300, 300, 64, True, True, 0), (384, 384, 64, True, False, 0),
    (577, 577, 128, True, False, 0), (128, 65, 128, False, False, 0), (130, 64, 64, False, False, 0), (192, 450, 128, False, False, 0), (192, 320, 64, False, True, 0), (448, 448, 128, False, False, 0),
    (196, 324, 128, True, False, 0), (512, 512, 128, True, False, 128)])
def test_one_q_block_per_workgroup_gives_the_same_bits(Nq, Nk, d, causal, token_major, block):
    blocks = -(-Nq // 64)
    few, many = 2, 800 // blocks + 8       # use_dq_split: at most 768 Q blocks with the mask, 512 without
    g = torch.Generator(device="cuda").manual_seed(Nq + Nk + d)
    rand = lambda n: torch.randn((1, many, n, d), generator=g, device="cuda").to(torch.bfloat16)
    Q, K, V, dO = rand(Nq), rand(Nk), rand(Nk), rand(Nq)
    lay = (lambda t: t.transpose(1, 2).contiguous()) if token_major else (lambda t: t.contiguous())
    params = lambda n: binding.SageParams(1, n, Nq, d, causal=causal, Nkv=Nk, token_major=token_major, bq=block, bkv=block)
    O, L = binding.sagebwd_fwd(lay(Q), lay(K), lay(V), params(many))
    want = binding.sagebwd_bwd(lay(Q), lay(K), lay(V), O, lay(dO), L, params(many))
    O2 = O[:, :, :few] if token_major else O[:, :few]
    got = binding.sagebwd_bwd(*(lay(t[:, :few]) for t in (Q, K, V)), O2.contiguous(), lay(dO[:, :few]), L[:, :few].contiguous(), params(few))
    torch.cuda.synchronize()
    for name, a, b in zip(("dQ", "dK", "dV"), got, want):
        b = b[:, :, :few] if token_major else b[:, :few]
        assert torch.isfinite(a.float()).all() and a.float().abs().max() > 0 and torch.equal(a, b), name


def test_psi_ds_past_the_caches_and_one_stage():
    """Tiles that do not fit the caches beside the tensors (12 heads of N = 6144 with the mask, and 6 of 8192, which take the form with one Q block per
    workgroup: loaded past them, the last heads first) against one head's; a walk of one stage."""
    d = 128
    g = torch.Generator(device="cuda").manual_seed(5)
    for heads, N in ((12, 6144), (6, 8192), (3, 64)):
        Q, K, V, dO = (torch.randn((1, heads, N, d), generator=g, device="cuda").to(torch.bfloat16) for _ in range(4))
        p = binding.SageParams(1, heads, N, d)
        O, L = binding.sagebwd_fwd(Q, K, V, p)
        dQ = binding.sagebwd_bwd(Q, K, V, O, dO, L, p)[0]
        one = binding.SageParams(1, 1, N, d)
        for h in (0, heads - 1):
            pick = lambda t: t[:, h:h + 1].contiguous()
            assert torch.equal(dQ[:, h:h + 1], binding.sagebwd_bwd(*(pick(t) for t in (Q, K, V, O, dO, L)), one)[0])
