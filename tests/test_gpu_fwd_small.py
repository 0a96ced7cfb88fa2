"""The forward's forms for calls that do not fill the machine, at the sizes where each can go wrong."""
import numpy as np
import pytest
import torch

import oracle
from paper_2603_02170_amd import binding, synth

from gpu_common import check_close, check_lse, to_np

pytestmark = pytest.mark.gpu


def _inputs(B, H, Nq, Nk, d, normed=False, q_offset=False):
    Q = synth.gaussian_inputs(Nq, d, sigma_qk=1.5, seed=11 * Nq + Nk, heads=B * H)[0]
    _, K, V, _ = synth.gaussian_inputs(Nk, d, sigma_qk=1.5, seed=Nk + d, heads=B * H)
    Q, K, V = (t.reshape(B, H, t.shape[2], d) for t in (Q, K, V))
    if normed:      # unit RMS: small logit scales, the conversion-free logits
        Q, K = (torch.nn.functional.rms_norm(t.float(), (d,)).to(torch.bfloat16) for t in (Q, K))
    if q_offset:
        Q = (Q.float() + torch.linspace(-2, 2, d)).to(torch.bfloat16)
    return Q, K, V


def _against_oracle(Q, K, V, p, heads):
    lay = (lambda t: t.permute(0, 2, 1, 3).contiguous()) if p.token_major else (lambda t: t)
    O, L = binding.sagebwd_fwd(*(lay(t).cuda() for t in (Q, K, V)), p)
    torch.cuda.synchronize()
    O, L = to_np(lay(O)), L.cpu().numpy()
    for b, h in heads:
        Or, Lr = oracle.forward_head(*(to_np(t[b, h]) for t in (Q, K, V)), causal=p.causal, k_smooth=p.k_smooth, q_smooth=p.q_smooth)
        check_close(f"O[{b},{h}]", O[b, h], Or)
        check_lse(f"LSE[{b},{h}]", L[b, h], Lr)


# Short caches, which the forms with codes in the workspace serve: one key, one block, a partial block, four blocks and just
# past them.  The kernel without (from 16 blocks on at d = 64 and 20 at d = 128, or about 512 blocks over all heads): its
# shortest caches and one key less, one workgroup per head and many with a ragged end, one key, 1 to 32 query rows, waves
# with several blocks and without any.
@pytest.mark.parametrize("B,H,Nq,Nk,d,k_smooth,token_major", [
    (1, 2, 1, 1, 128, True, False), (1, 2, 1, 64, 64, True, False), (1, 3, 5, 200, 64, False, True), (1, 2, 32, 256, 128, True, False),
    (1, 2, 3, 257, 128, True, False), (2, 3, 7, 2049, 64, True, True), (1, 1, 31, 8192, 128, True, False), (8, 32, 1, 640, 128, True, False), (1, 2, 9, 1024, 128, True, False), (1, 2, 2, 1023, 64, False, True),
    (1, 2, 4, 961, 64, True, False), (1, 2, 4, 960, 64, True, False), (1, 2, 4, 1473, 128, True, False), (1, 2, 4, 1472, 128, False, False),
    (32, 32, 1, 1, 64, True, False), (16, 32, 5, 100, 128, False, True),
    (4, 32, 32, 1100, 64, True, False), (1, 1, 32, 20000, 64, True, False)])
def test_decode(B, H, Nq, Nk, d, k_smooth, token_major):
    Q, K, V = _inputs(B, H, Nq, Nk, d)
    p = binding.SageParams(B, H, Nq, d, causal=False, k_smooth=k_smooth, Nkv=Nk, token_major=token_major)
    _against_oracle(Q, K, V, p, {(0, 0), (B - 1, H - 1)})


# The join of partial results: one past a wave's 64, one more than the groups of threads (8 at d = 128, 16 at d = 64), fewer;
# blocks per wave: one and more, a last workgroup of one block; the line at 20 blocks and at 512
@pytest.mark.parametrize("B,H,Nq,Nk,d,k_smooth", [
    (1, 1, 2, 64 * 257, 128, True), (1, 1, 32, 64 * 257, 64, False), (1, 2, 3, 64 * 33, 128, False), (1, 2, 3, 64 * 65, 64, True),
    (2, 32, 4, 64 * 32, 128, True), (1, 32, 2, 64 * 65 - 5, 128, True), (4, 32, 1, 64 * 37, 64, True), (4, 32, 17, 64 * 37 - 63, 128, False),
    (1, 2, 1, 64 * 19, 128, True), (1, 2, 1, 64 * 19 + 1, 128, True), (8, 32, 2, 65, 128, True), (8, 32, 2, 64, 128, True),
    # one workgroup per head between one and two rounds of them, two where the walks are long; two blocks for each wave; one and
    # two blocks with K-smoothing (codes) and without
    (4, 45, 3, 64 * 12 - 3, 64, True), (4, 45, 2, 64 * 32 - 40, 128, True), (5, 45, 1, 64 * 9 + 1, 128, False), (8, 16, 32, 64 * 8 - 1, 64, False),
    (5, 16, 4, 64 * 8, 128, True), (16, 32, 2, 64, 128, False), (16, 32, 2, 64, 128, True), (6, 50, 2, 128, 128, True), (8, 50, 2, 127, 128, True)])
def test_decode_splits(B, H, Nq, Nk, d, k_smooth):
    Q, K, V = _inputs(B, H, Nq, Nk, d)
    _against_oracle(Q, K, V, binding.SageParams(B, H, Nq, d, causal=False, k_smooth=k_smooth, Nkv=Nk), {(0, 0), (B - 1, H - 1)})


@pytest.mark.parametrize("Nk", [200, 1100])       # codes in the workspace; a decoding step
def test_decode_leaves_the_quantised_tensors_for_those_who_can_read_them(Nk):
    """Codes and scales after a forward on the full workspace, and a backward that shares them."""
    Q, K, V = (t.cuda() for t in _inputs(1, 2, 9, Nk, 64))
    p = binding.SageParams(1, 2, 9, 64, causal=False, Nkv=Nk)
    ws, ws2 = binding.alloc_workspace(p), binding.alloc_workspace(p)
    O, L = binding.sagebwd_fwd(Q, K, V, p, ws)
    binding.sagebwd_quantize(Q, K, V, p, ws2)
    for which in (binding.TENSOR_Q, binding.TENSOR_K, binding.TENSOR_V):
        for a, b in zip(binding.sagebwd_export_quantized(p, ws, which), binding.sagebwd_export_quantized(p, ws2, which)):
            assert torch.equal(a, b), which
    dO = torch.ones_like(O)
    ref = binding.sagebwd_bwd(Q, K, V, O, dO, L, p)
    ps = binding.SageParams(1, 2, 9, 64, causal=False, Nkv=Nk, share_quantized=True)
    wss = binding.alloc_workspace(ps)
    Os, Ls = binding.sagebwd_fwd(Q, K, V, ps, wss)
    assert torch.equal(O, Os) and torch.equal(L, Ls)
    for a, b in zip(ref, binding.sagebwd_bwd(Q, K, V, Os, dO, Ls, ps, wss)):
        assert torch.equal(a, b)


# eight tiles for four splits, a number of tiles the splits do not divide, nine tiles (the last split gets none) with and
# without the mask, query rows that do not exist, both ring depths, Q-smoothing's biases in the ring
@pytest.mark.parametrize("Nq,Nk,d,causal,q_smooth", [(64, 512, 128, False, False), (100, 868, 64, True, False), (192, 580, 128, False, True),
                                                     (33, 609, 64, False, True), (256, 1024, 128, True, False), (64, 4160, 128, True, True),
                                                     (64, 576, 128, True, False), (40, 530, 64, False, False), (64, 576, 64, True, True)])
def test_split_keys(Nq, Nk, d, causal, q_smooth):
    Q, K, V = _inputs(1, 2, Nq, Nk, d, normed=not q_smooth, q_offset=q_smooth)
    _against_oracle(Q, K, V, binding.SageParams(1, 2, Nq, d, causal=causal, q_smooth=q_smooth, Nkv=Nk), {(0, 0), (0, 1)})


# one tile, two, a partial last block, the corrections of the bias every eight tiles, the conversion-free logits and the
# converting ones: a head alone (two waves per 32 queries) and in a call that fills the machine (one wave)
@pytest.mark.parametrize("N,d,causal,normed,q_smooth", [(64, 128, True, True, False), (128, 64, False, False, False), (200, 128, True, True, False),
                                                        (577, 64, True, True, False), (640, 128, False, True, False), (320, 128, True, False, True)])
def test_two_waves_per_query_group_give_the_same_bits(N, d, causal, normed, q_smooth):
    heads = -(-1024 // (-(-N // 32))) + 8
    Q, K, V = (t.cuda() for t in _inputs(1, heads, N, N, d, normed=normed, q_offset=q_smooth))
    O, L = binding.sagebwd_fwd(Q, K, V, binding.SageParams(1, heads, N, d, causal=causal, q_smooth=q_smooth))
    p1 = binding.SageParams(1, 1, N, d, causal=causal, q_smooth=q_smooth)
    for h in (0, heads - 1):
        O1, L1 = binding.sagebwd_fwd(*(t[:, h:h + 1].contiguous() for t in (Q, K, V)), p1)
        torch.cuda.synchronize()
        assert torch.equal(O1[0, 0], O[0, h]) and torch.equal(L1[0, 0], L[0, h]), h
    assert np.isfinite(to_np(O)).all()


# More keys than queries: the division of the keys over waves depends on how many heads the call has.  Then O differs by
# at most its two bf16 roundings (2^-9 each) in the 2-norm, and LSE by what the biased logits cost (1e7 c 2^-24 in log2
# units, c about 1e-4 for such inputs).  Fewer than twice as many keys: the same bits.
@pytest.mark.parametrize("heads,Nq,Nk,d,causal,same", [(64, 1, 8192, 128, False, False), (128, 512, 1100, 128, False, False), (128, 128, 576, 64, True, False),
                                                       (1024, 20, 64, 64, False, False), (64, 512, 960, 128, True, True), (70, 100, 150, 64, False, True)])
def test_a_head_alone_and_in_a_batch(heads, Nq, Nk, d, causal, same):
    Q, K, V = (t.cuda() for t in _inputs(1, heads, Nq, Nk, d, normed=True))
    O, L = binding.sagebwd_fwd(Q, K, V, binding.SageParams(1, heads, Nq, d, causal=causal, Nkv=Nk))
    again = binding.sagebwd_fwd(Q, K, V, binding.SageParams(1, heads, Nq, d, causal=causal, Nkv=Nk))
    assert torch.equal(O, again[0]) and torch.equal(L, again[1])
    for h in (0, heads - 1):
        O1, L1 = binding.sagebwd_fwd(*(t[:, h:h + 1].contiguous() for t in (Q, K, V)), binding.SageParams(1, 1, Nq, d, causal=causal, Nkv=Nk))
        torch.cuda.synchronize()
        if same:
            assert torch.equal(O1[0, 0], O[0, h]) and torch.equal(L1[0, 0], L[0, h])
        else:
            a, b = O[0, h].double(), O1[0, 0].double()
            assert float((a - b).norm()) <= 2 ** -8 * float(b.norm())
            assert float((L[0, h] - L1[0, 0]).abs().max()) <= 1e-4


def _from_the_stored_codes(p, Q, K, V):
    """The forward in float64 from the codes and scales that the pre-pass stores (its quantiser of P~ included)."""
    ws = binding.alloc_workspace(p)
    binding.sagebwd_quantize(Q, K, V, p, ws)
    (q, sq), (k, sk), (v, sv) = ([t.cpu().numpy().astype(np.float64) for t in binding.sagebwd_export_quantized(p, ws, w)]
                                 for w in (binding.TENSOR_Q, binding.TENSOR_K, binding.TENSOR_V))
    nk, nblk = p.kv_len, k.shape[2] // 64
    O = np.zeros((p.B, p.H, p.N, p.d))
    for b in range(p.B):
        for h in range(p.H):
            o = l = 0.0
            for j in range(nblk):
                sl = slice(64 * j, min(64 * j + 64, nk))
                s = q[b, h, :p.N] @ k[b, h, sl].T * (sq[b, h, 0] * sk[b, h, j] / np.sqrt(p.d))
                m = s.max(1, keepdims=True)
                e = 127.0 * np.exp(s - m)
                w = np.exp(m)                                   # (logits of this test are small)
                o = o + w * sv[b, h, j] * (np.rint(e) @ v[b, h, sl])
                l = l + w * e.sum(1, keepdims=True)
            O[b, h] = o / l
    return O


# what a value that is not a number, an infinite factor 127 / max|x| or a block of zeros becomes is the pre-pass's choice
# (a code within +-127): a decoding step, which keeps its codes in registers, has to take the same one
@pytest.mark.parametrize("what", ["plain", "nan_v", "nan_k", "nan_q", "tiny_v", "tiny_some_v", "zero_v"])
@pytest.mark.parametrize("Nq", [5, 40])       # a decoding step; the same through the workspace
def test_codes_of_exceptional_blocks(what, Nq):
    Q, K, V = (t.clone() for t in _inputs(1, 2, Nq, 1100, 64, normed=True))
    if what == "nan_v":
        V[0, :, 70:80, 3] = float("nan")
    elif what == "nan_k":
        K[0, :, 130, 7] = float("nan")
    elif what == "nan_q":
        Q[0, :, 1, 9] = float("nan")
    elif what == "tiny_v":
        V = (V.float() * 2.0 ** -126).to(torch.bfloat16)        # 127 / max|v| is infinite
        V[..., 5] = 0
    elif what == "tiny_some_v":
        V[0, :, 64:128] = (V[0, :, 64:128].float() * 2.0 ** -126).to(torch.bfloat16)
    elif what == "zero_v":
        V[0, :, 64:640] = 0
    Q, K, V = (t.cuda() for t in (Q, K, V))
    p = binding.SageParams(1, 2, Nq, 64, causal=False, k_smooth=False, Nkv=1100)
    O, _ = binding.sagebwd_fwd(Q, K, V, p)
    ref = _from_the_stored_codes(p, Q, K, V)
    O = O.float().cpu().numpy().astype(np.float64)
    # bf16 rounding is 2^-9 of a value; single codes of P~ may fall to the other side of a step
    assert np.linalg.norm(O - ref) <= 6e-3 * np.linalg.norm(ref), np.linalg.norm(O - ref) / np.linalg.norm(ref)
