"""Heads of one and two blocks in every form that serves them: one launch, and the separate launches with one, two and four waves per 32
queries, or one and two KV blocks per workgroup.  (Outputs in the memory of inputs keep a call from the forms of one launch.)"""
import pytest
import torch

from paper_2603_02170_amd import binding

pytestmark = pytest.mark.gpu


def _bits(t):
    return t.contiguous().view(torch.int16 if t.dtype == torch.bfloat16 else torch.int32 if t.dtype == torch.float32 else torch.int8)


def _inputs(heads, Nq, Nk, d, normed):
    """Logits whose maximum over the second key block lies above that over the first by nothing up to many times the step at which the
    running reference is raised, more with each head (through a direction that its keys and all queries share)."""
    g = torch.Generator(device="cuda").manual_seed(1000 * Nq + Nk + d)
    Q, K, V, dO = (torch.randn((1, heads, n, d), generator=g, device="cuda") for n in (Nq, Nk, Nk, Nq))
    u = torch.randn(d, generator=g, device="cuda").sign()
    Q += 0.7 * u
    K[:, :, 64:] += u * torch.linspace(0, 2, heads, device="cuda")[None, :, None, None]
    if normed:      # unit RMS: small logit scales, the conversion-free logits
        Q, K = (x * torch.rsqrt(x.square().mean(-1, keepdim=True)) for x in (Q, K))
    else:
        Q[0, ::2] *= 40
    return [t.to(torch.bfloat16) for t in (Q, K, V, dO)]


def _separate(Q, K, V, p, ws=None):
    """The forward in separate launches: O begins in the last row of V."""
    buf = torch.cat([V.reshape(-1), torch.zeros(Q.numel(), dtype=V.dtype, device="cuda")])
    v, o = buf[:V.numel()].view(V.shape), buf[V.numel() - p.d:V.numel() - p.d + Q.numel()].view(Q.shape)
    return binding.sagebwd_fwd(Q, K, v, p, ws, o)


# a full block, one row more and less, two, a partial second one, more and fewer queries than keys, the mask with a shift, three Q blocks
SHAPES = [(64, 64, 128, True), (64, 64, 64, False), (33, 33, 64, False), (65, 65, 128, True), (100, 100, 64, True), (128, 128, 64, True), (128, 128, 128, False),
          (64, 128, 128, True), (40, 104, 64, True), (33, 128, 128, False), (192, 64, 64, False), (150, 40, 128, False)]


@pytest.mark.parametrize("normed", [True, False])
@pytest.mark.parametrize("Nq,Nk,d,causal", SHAPES)
def test_forward(Nq, Nk, d, causal, normed):
    blocks = -(-Nq // 64)
    many = 1024 // blocks + 16           # one wave per 32 queries; two workgroups of two waves at d = 64
    Q, K, V, _ = _inputs(many, Nq, Nk, d, normed)
    kw = dict(causal=causal, Nkv=Nk, k_smooth=normed)
    O, L = _separate(Q, K, V, binding.SageParams(1, many, Nq, d, **kw))
    assert torch.isfinite(O.float()).all() and torch.isfinite(L).all()
    for n in (2, 257 // blocks + 8, many):
        part, p = [t[:, -n:].contiguous() for t in (Q, K, V)], binding.SageParams(1, n, Nq, d, **kw)
        for o, l in (_separate(*part, p), binding.sagebwd_fwd(*part, p)):
            torch.cuda.synchronize()
            assert torch.equal(o, O[:, -n:]) and torch.equal(l, L[:, -n:]), n


@pytest.mark.parametrize("Nq,Nk,d,causal", SHAPES)
def test_backward(Nq, Nk, d, causal):
    if Nq > 128:
        Nq = 128
    nq, nk = -(-Nq // 64), -(-Nk // 64)
    heads = 512 // nk + 9
    Q, K, V, dO = _inputs(heads, Nq, Nk, d, True)
    kw = dict(causal=causal, Nkv=Nk)
    O, L = binding.sagebwd_fwd(Q, K, V, binding.SageParams(1, heads, Nq, d, **kw))
    head = nq * (nk + 3) * 4096          # bytes of psi(dS) of a head
    # in one launch where that is taken; all heads but one together; one head at a time
    got = [binding.sagebwd_bwd(Q, K, V, O, dO, L, binding.SageParams(1, heads, Nq, d, scratch_budget=b, **kw)) for b in (0, (heads - 1) * head, 1)]
    few = binding.sagebwd_bwd(*(t[:, :3].contiguous() for t in (Q, K, V, O, dO)), L[:, :3].contiguous(), binding.SageParams(1, 3, Nq, d, **kw))
    torch.cuda.synchronize()
    for name, a, b, c, f in zip(("dQ", "dK", "dV"), *got, few):
        assert torch.isfinite(a.float()).all() and torch.equal(a, b) and torch.equal(a, c) and torch.equal(a[:, :3], f), name


@pytest.mark.parametrize("Nq,Nk,d,causal", [(64, 64, 128, True), (128, 128, 64, True), (100, 100, 128, True), (33, 128, 64, False), (128, 50, 128, False), (64, 128, 128, True)])
def test_psi_of_dS(Nq, Nk, d, causal):
    heads = 3
    Q, K, V, dO = _inputs(heads, Nq, Nk, d, True)
    p = binding.SageParams(1, heads, Nq, d, causal=causal, Nkv=Nk)
    left = []
    for separate in (False, True):
        ws = binding.alloc_workspace(p)
        ws.fill_(0x5a)
        O, L = binding.sagebwd_fwd(Q, K, V, p, ws)
        buf = torch.cat([Q.reshape(-1), torch.zeros(d, dtype=Q.dtype, device="cuda")])
        q, dq = buf[:Q.numel()].view(Q.shape), (buf[d:] if separate else torch.empty_like(Q).view(-1)).view(Q.shape)
        binding.sagebwd_bwd(q, K, V, O, dO, L, p, ws, dq, torch.empty_like(K), torch.empty_like(V))
        left.append([dq.clone()] + [t for h in range(heads) for t in binding.sagebwd_export_ds(p, ws, h)])
    torch.cuda.synchronize()
    assert left[0][1].abs().max() > 0
    for n, (a, b) in enumerate(zip(*left)):
        assert torch.equal(_bits(a), _bits(b)), n


@pytest.mark.parametrize("Nq,Nk,d", [(64, 64, 128), (100, 100, 64), (33, 128, 128)])
def test_gradients_into_tensors_that_are_not_16_byte_aligned(Nq, Nk, d):
    """Gradients leave in 16-byte pieces; a caller's tensors need not start at such an address."""
    heads = 5
    Q, K, V, dO = _inputs(heads, Nq, Nk, d, True)
    p = binding.SageParams(1, heads, Nq, d, causal=False, Nkv=Nk)
    O, L = binding.sagebwd_fwd(Q, K, V, p)
    want = binding.sagebwd_bwd(Q, K, V, O, dO, L, p)
    for offset in (2, 4):
        into = [torch.empty(t.numel() + offset, dtype=t.dtype, device="cuda")[offset:].view(t.shape) for t in (Q, K, V)]
        binding.sagebwd_bwd(Q, K, V, O, dO, L, p, None, *into)
        torch.cuda.synchronize()
        for a, b in zip(into, want):
            assert torch.equal(a, b), offset
