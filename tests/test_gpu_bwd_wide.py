"""The backward with four KV blocks per workgroup gives the bits of the forms that a head alone takes."""
import pytest
import torch

from paper_2603_02170_amd import binding, synth

pytestmark = pytest.mark.gpu


# three to ten KV blocks (workgroups with idle waves; also one and two, which the form with two blocks serves), one Q block and more, whole and partial last blocks of either side, the mask
# with and without a shift (the diagonal of the four blocks lies in different intervals), numerics blocks of 128 in either direction
# (pairs of blocks of which one does not exist, is not visible, or lies in the next workgroup; odd and even Q block counts)
# and Q-smoothing (the bias of every block's keys, the sums for the bias branch of dK)
@pytest.mark.parametrize("bq,bkv,q_smooth", [(0, 0, False), (0, 0, True), (64, 128, False), (128, 64, False), (128, 128, False)])
@pytest.mark.parametrize("Nq,Nk,causal", [(64, 64, True), (1, 100, False), (50, 600, False), (100, 228, True), (256, 256, True), (300, 300, True),
                                          (640, 640, True), (200, 321, False), (448, 70, False), (64, 512, True), (130, 450, True),
                                          (192, 192, True), (1, 170, False), (64, 192, False), (448, 140, False)])
def test_four_kv_blocks_per_workgroup_give_the_same_bits(Nq, Nk, causal, bq, bkv, q_smooth):
    d, nblk = 128, -(-Nk // 64)
    heads = 1024 // nblk + 9            # enough for four blocks per workgroup from three KV blocks on (bwd_wide_is_faster)
    g = torch.Generator(device="cuda").manual_seed(1000 * Nq + Nk)
    rand = lambda n, s: (torch.randn((1, heads, n, d), generator=g, device="cuda") * s).to(torch.bfloat16)
    Q, K, V, dO = rand(Nq, 1.5), rand(Nk, 1.5), rand(Nk, 1.0), rand(Nq, 1.0)
    kw = dict(causal=causal, Nkv=Nk, bq=bq, bkv=bkv, q_smooth=q_smooth)
    p, p1 = binding.SageParams(1, heads, Nq, d, **kw), binding.SageParams(1, 1, Nq, d, **kw)
    O, L = binding.sagebwd_fwd(Q, K, V, p)
    many = binding.sagebwd_bwd(Q, K, V, O, dO, L, p)
    for h in (0, heads // 2, heads - 1):
        sl = slice(h, h + 1)
        one = binding.sagebwd_bwd(*(t[:, sl].contiguous() for t in (Q, K, V, O, dO)), L[:, sl].contiguous(), p1)
        torch.cuda.synchronize()
        for a, b, name in zip(many, one, ("dQ", "dK", "dV")):
            assert torch.isfinite(b.float()).all()
            assert torch.equal(a[:, sl], b), (h, name)


@pytest.mark.parametrize("Nq,Nk,causal", [(200, 321, False), (640, 640, True), (1, 100, False)])
def test_token_major_tensors(Nq, Nk, causal):
    heads, d = 1024 // (-(-Nk // 64)) + 9, 128
    g = torch.Generator(device="cuda").manual_seed(Nq + Nk)
    rand = lambda n: torch.randn((1, heads, n, d), generator=g, device="cuda").to(torch.bfloat16)
    Q, K, V, dO = rand(Nq), rand(Nk), rand(Nk), rand(Nq)
    got = []
    for tm in (False, True):
        p = binding.SageParams(1, heads, Nq, d, causal=causal, Nkv=Nk, token_major=tm)
        q, k, v, do = (t.transpose(1, 2).contiguous() if tm else t for t in (Q, K, V, dO))
        O, L = binding.sagebwd_fwd(q, k, v, p)
        grads = binding.sagebwd_bwd(q, k, v, O, do, L, p)
        torch.cuda.synchronize()
        got.append([t.transpose(1, 2) if tm else t for t in grads])
    for a, b in zip(*got):
        assert torch.equal(a, b)


# scratch for nine heads of 32 workgroups each: two groups of eight (a round each) instead of nine and seven; for one head; for five of
# three workgroups, where more heads never take more rounds; for four of seven heads, whose psi(dS) is then loaded past the caches
# (ds_traffic), the last heads first, that of the other three through them, and stored past them as well where all seven are one group
@pytest.mark.parametrize("heads,N,fit", [(16, 8192, 9), (3, 2048, 1), (12, 640, 5), (7, 8192, 4)])
def test_groups_of_heads_without_the_mask(heads, N, fit):
    d, nblk = 128, N // 64
    g = torch.Generator(device="cuda").manual_seed(N)
    Q, K, V, dO = (torch.randn((1, heads, N, d), generator=g, device="cuda").to(torch.bfloat16) for _ in range(4))
    p = binding.SageParams(1, heads, N, d, causal=False)
    small = binding.SageParams(1, heads, N, d, causal=False, scratch_budget=fit * nblk * (nblk + 3) * 4096)
    O, L = binding.sagebwd_fwd(Q, K, V, p)
    whole, parts = binding.sagebwd_bwd(Q, K, V, O, dO, L, p), binding.sagebwd_bwd(Q, K, V, O, dO, L, small)
    torch.cuda.synchronize()
    for a, b in zip(whole, parts):
        assert torch.equal(a, b)


def test_gradients_into_tensors_that_are_not_16_byte_aligned():
    """dK and dV leave in 16-byte pieces; a caller's tensors need not start at such an address."""
    heads, N, d = 140, 256, 128
    g = torch.Generator(device="cuda").manual_seed(5)
    Q, K, V, dO = (torch.randn((1, heads, N, d), generator=g, device="cuda").to(torch.bfloat16) for _ in range(4))
    p = binding.SageParams(1, heads, N, d, causal=False)
    O, L = binding.sagebwd_fwd(Q, K, V, p)
    want = binding.sagebwd_bwd(Q, K, V, O, dO, L, p)
    shifted = [torch.empty(Q.numel() + 4, dtype=torch.bfloat16, device="cuda")[4:].view(Q.shape) for _ in range(3)]
    got = binding.sagebwd_bwd(Q, K, V, O, dO, L, p, None, *shifted)
    torch.cuda.synchronize()
    for a, b, s in zip(got, want, shifted):
        assert a.data_ptr() == s.data_ptr() and a.data_ptr() % 16 == 8 and torch.equal(a, b)
