"""The autograd wrapper returns the bits of the two direct calls and wires the gradients to Q, K, V."""
import threading

import pytest
import torch
from torch.utils.checkpoint import checkpoint

from paper_2603_02170_amd import binding, synth
from paper_2603_02170_amd.autograd import sage_attention

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,Nk,d,causal,token_major,share", [(192, 192, 64, True, False, False), (100, 228, 128, True, False, True),
                                                             (256, 256, 128, False, True, True), (77, 150, 64, False, True, False)])
def test_autograd_wrapper_gives_the_bits_of_the_direct_calls(N, Nk, d, causal, token_major, share):
    H = 3
    Q, _, _, dO = synth.gaussian_inputs(N, d, sigma_qk=1.5, seed=N + d, heads=H)
    _, K, V, _ = synth.gaussian_inputs(Nk, d, sigma_qk=1.5, seed=N + d + 1, heads=H)
    Q, K, V, dO = (t.cuda() for t in (Q, K, V, dO))
    if token_major:
        Q, K, V, dO = (t.permute(0, 2, 1, 3).contiguous() for t in (Q, K, V, dO))
    p = binding.SageParams(1, H, N, d, causal=causal, token_major=token_major, Nkv=0 if Nk == N else Nk)
    O, L = binding.sagebwd_fwd(Q, K, V, p)
    dQ, dK, dV = binding.sagebwd_bwd(Q, K, V, O, dO, L, p)
    q, k, v = (t.clone().requires_grad_(True) for t in (Q, K, V))
    o, lse = sage_attention(q, k, v, causal=causal, token_major=token_major, share_quantized=share, return_lse=True)
    assert not lse.requires_grad
    o.backward(dO)
    torch.cuda.synchronize()
    assert torch.equal(o.detach(), O) and torch.equal(lse, L)
    assert torch.equal(q.grad, dQ) and torch.equal(k.grad, dK) and torch.equal(v.grad, dV)


def test_autograd_wrapper_in_a_training_step():
    """A projection trained through the INT8 attention: the loss falls (the gradients point downhill)."""
    torch.manual_seed(0)
    B, H, N, d = 1, 2, 128, 64
    x = torch.randn(B, H, N, d, device="cuda")
    target = torch.randn(B, H, N, d, device="cuda")
    W = (torch.eye(d, device="cuda") + 0.05 * torch.randn(d, d, device="cuda")).requires_grad_(True)
    losses = []
    for _ in range(12):
        h = (x @ W).to(torch.bfloat16)
        o = sage_attention(h, h, h, causal=True)
        loss = ((o.float() - target) ** 2).mean()
        loss.backward()
        with torch.no_grad():
            W -= 0.5 * W.grad
            W.grad = None
        losses.append(float(loss.detach()))
    assert losses[-1] < 0.97 * losses[0], losses


def test_a_causal_flag_that_is_neither_0_nor_1_is_refused():
    x = [torch.zeros(1, 1, 64, 64, dtype=torch.bfloat16, device="cuda") for _ in range(3)]
    for call in (lambda: sage_attention(*x, causal=2), lambda: binding.sagebwd_fwd(*x, binding.SageParams(1, 1, 64, 64, causal=2))):
        with pytest.raises(binding.SageError) as e:
            call()
        assert e.value.status == -1


def _case(N=150, d=64, seed=3):
    Q, K, V, dO = (t.cuda() for t in synth.gaussian_inputs(N, d, sigma_qk=1.5, seed=seed, heads=3))
    p = binding.SageParams(1, 3, N, d, causal=True)
    O, L = binding.sagebwd_fwd(Q, K, V, p)
    return (Q, K, V), dO, O, binding.sagebwd_bwd(Q, K, V, O, dO, L, p)


def _leaves(ts):
    return [t.clone().requires_grad_() for t in ts]


@pytest.mark.parametrize("share", [False, True])
def test_a_retained_graph_gives_the_same_gradients_again(share):
    x, dO, _, ref = _case()
    x = _leaves(x)
    o = sage_attention(*x, share_quantized=share)
    for k in range(3):      # (with `share` the first backward uses up the forward's workspace)
        got = torch.autograd.grad(o, x, dO, retain_graph=k < 2)
        assert all(torch.equal(a, b) for a, b in zip(got, ref)), k
    with pytest.raises(RuntimeError, match="second time"):
        torch.autograd.grad(o, x, dO)


@pytest.mark.parametrize("share", [False, True])
def test_saved_tensor_hooks_see_what_the_node_keeps(share):
    x, dO, o_ref, ref = _case()
    x = _leaves(x)
    packed = []

    def pack(t):
        packed.append(t.shape)
        return t.cpu()

    with torch.autograd.graph.saved_tensors_hooks(pack, lambda t: t.cuda()):
        o = sage_attention(*x, share_quantized=share)
    assert len(packed) == 5 and torch.equal(o.detach(), o_ref)          # Q, K, V, L and O
    got = torch.autograd.grad(o, x, dO)
    assert all(torch.equal(a, b) for a, b in zip(got, ref))


@pytest.mark.parametrize("reentrant", [False, True])
def test_under_checkpointing(reentrant):
    x, dO, _, ref = _case()
    x = _leaves(x)
    o = checkpoint(lambda q, k, v: sage_attention(q, k, v) * 1.0, *x, use_reentrant=reentrant)
    o.backward(dO)
    assert all(torch.equal(t.grad, b) for t, b in zip(x, ref))


def test_operands_and_gradients_that_are_not_contiguous():
    x, dO, o_ref, ref = _case()
    x = _leaves(x)
    strided = [t.transpose(1, 2).contiguous().transpose(1, 2) for t in x]       # same values, token-major strides
    assert not any(t.is_contiguous() for t in strided)
    o = sage_attention(*strided)
    assert torch.equal(o.detach(), o_ref)
    o.backward(dO.transpose(1, 2).contiguous().transpose(1, 2))
    assert all(torch.equal(t.grad, b) for t, b in zip(x, ref))
    # a gradient of stride zero
    y = _leaves([t.detach() for t in x])
    a = torch.autograd.grad(sage_attention(*y).sum(), y)
    b = torch.autograd.grad(sage_attention(*y), y, torch.ones_like(dO))
    assert all(torch.equal(s, t) for s, t in zip(a, b))


@pytest.mark.parametrize("wanted", [(0,), (1,), (2,), (0, 2), ()])
def test_gradients_of_some_operands_only(wanted):
    x, dO, o_ref, ref = _case()
    x = [t.clone().requires_grad_(k in wanted) for k, t in enumerate(x)]
    o = sage_attention(*x)
    assert torch.equal(o.detach(), o_ref) and o.requires_grad == bool(wanted)
    if wanted:
        o.backward(dO)
    for k in range(3):
        assert torch.equal(x[k].grad, ref[k]) if k in wanted else x[k].grad is None
    with torch.no_grad():
        assert not sage_attention(*x).requires_grad


def test_an_operand_changed_in_place_is_noticed():
    x, dO, _, _ = _case()
    for what in (0, 1, 2, 3):
        leaves = _leaves(x)
        y = [t * 1.0 for t in leaves]
        o = sage_attention(*y)
        with torch.no_grad():
            (y + [o])[what].add_(1.0)
        with pytest.raises(RuntimeError, match="modified by an inplace operation"):
            o.backward(dO)


@pytest.mark.parametrize("share", [False, True])
def test_forward_and_backward_on_a_second_stream(share):
    x, dO, o_ref, ref = _case()
    x = _leaves(x)
    torch.cuda.synchronize()
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        o = sage_attention(*x, share_quantized=share)
    junk = [torch.full_like(dO, 7.0) for _ in range(4)]       # allocations of the default stream meanwhile
    got = torch.autograd.grad(o, x, dO)                       # the engine runs the node on the forward's stream
    torch.cuda.synchronize()
    assert torch.equal(o.detach(), o_ref) and all(torch.equal(a, b) for a, b in zip(got, ref))
    assert all(bool((t == 7.0).all()) for t in junk)


def test_several_threads_at_once():
    cases = [_case(N=100 + 64 * k, seed=k) for k in range(4)]
    torch.cuda.synchronize()
    bad = []

    def work(k):
        x, dO, o_ref, ref = cases[k]
        with torch.cuda.stream(torch.cuda.Stream()):
            for share in (False, True, False, True):
                y = _leaves(x)
                o = sage_attention(*y, share_quantized=share)
                got = torch.autograd.grad(o, y, dO)
                torch.cuda.current_stream().synchronize()
                if not (torch.equal(o.detach(), o_ref) and all(torch.equal(a, b) for a, b in zip(got, ref))):
                    bad.append((k, share))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad


def test_dual_tensors_on_the_gpu_are_refused():
    import torch.autograd.forward_ad as fwAD
    x, _, _, _ = _case()
    with fwAD.dual_level(), pytest.raises(NotImplementedError):
        sage_attention(fwAD.make_dual(x[0], torch.ones_like(x[0])), x[1], x[2])
    with pytest.raises(RuntimeError):
        torch.vmap(lambda a: sage_attention(a, x[1], x[2]))(torch.stack([x[0], x[0]]))
