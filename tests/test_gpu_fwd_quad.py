"""The forward's form with four waves per 32 queries gives the bits of the forms with two waves and with one."""
import pytest
import torch

from paper_2603_02170_amd import binding

pytestmark = pytest.mark.gpu


# two tiles and three (a last pair of one tile), whole and partial last blocks, the first and second pair inside the unrolled loop and past
# it, the corrections of the bias every eight tiles, more keys than queries under the mask, conversion-free logits and converting ones, Q-smoothing;
# a row of one visible key
@pytest.mark.parametrize("Nq,Nk,d,causal,normed,q_smooth", [
    (65, 65, 128, True, True, False), (128, 128, 64, False, True, False), (192, 192, 128, False, False, False), (256, 256, 128, True, True, False),
    (300, 300, 64, True, False, False), (384, 384, 128, True, True, False), (449, 449, 64, True, True, False), (512, 512, 128, False, True, True), (577, 577, 128, True, False, True),
    (600, 600, 64, False, True, True), (640, 704, 128, True, True, False), (1100, 1100, 128, True, True, False), (1088, 1088, 64, True, True, False),
    # without the mask, an odd number of blocks of the calls that take it (fwd_quad_is_faster)
    (832, 832, 128, False, True, False), (813, 813, 64, False, False, False), (704, 704, 128, False, True, True)])
def test_four_waves_per_query_group_give_the_same_bits(Nq, Nk, d, causal, normed, q_smooth):
    blocks = -(-Nq // 64)
    heads = [2, 257 // blocks + 8, 1024 // blocks + 8]       # four waves, two, one (use_fwd_quad, use_fwd_pair)
    assert heads[0] * blocks <= 256 < heads[1] * blocks <= 512 < heads[2] * blocks
    g = torch.Generator(device="cuda").manual_seed(Nq + d)
    rand = lambda n: torch.randn((1, heads[2], n, d), generator=g, device="cuda")
    Q, K, V = rand(Nq) * 1.5, rand(Nk) * 1.5, rand(Nk)
    if normed:      # unit RMS: small logit scales, the conversion-free logits
        Q, K = (torch.nn.functional.rms_norm(t, (d,)) for t in (Q, K))
    if q_smooth:
        Q = Q + torch.linspace(-2, 2, d, device="cuda")
    Q, K, V = (t.to(torch.bfloat16) for t in (Q, K, V))
    got = []
    for n in heads:
        p = binding.SageParams(1, n, Nq, d, causal=causal, q_smooth=q_smooth, Nkv=Nk)
        got.append(binding.sagebwd_fwd(*(t[:, :n].contiguous() for t in (Q, K, V)), p))
    torch.cuda.synchronize()
    O, L = got[2]
    assert torch.isfinite(O.float()).all() and torch.isfinite(L).all()
    for o, l in got[:2]:
        assert torch.equal(o, O[:, :o.shape[1]]) and torch.equal(l, L[:, :l.shape[1]])


def test_a_second_round_of_workgroups_under_the_mask():
    """d = 128, long walks: more workgroups than CUs; against two waves per 32 queries (token-major tensors, whose rows lie elsewhere) and one."""
    N, d = 2048, 128
    g = torch.Generator(device="cuda").manual_seed(3)
    Q, K, V = (torch.randn((1, 40, N, d), generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    got = []
    for n in (12, 16, 40):
        tm = n == 16
        q, k, v = ((t[:, :n].transpose(1, 2) if tm else t[:, :n]).contiguous() for t in (Q, K, V))
        O, L = binding.sagebwd_fwd(q, k, v, binding.SageParams(1, n, N, d, token_major=tm))
        got.append((O.transpose(1, 2) if tm else O, L))
    torch.cuda.synchronize()
    for o, l in got[:2]:
        assert torch.equal(o, got[2][0][:, :o.shape[1]]) and torch.equal(l, got[2][1][:, :l.shape[1]])
