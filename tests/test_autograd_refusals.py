"""What sage_attention cannot differentiate it refuses, before it looks at shapes and devices (no GPU needed)."""
import os

import pytest
import torch
import torch.autograd.forward_ad as fwAD

from paper_2603_02170_amd import build
from paper_2603_02170_amd.autograd import sage_attention


@pytest.fixture(scope="module", autouse=True)
def built():
    if not os.path.exists(build.HOST):
        build.build(verbose=False)


def _qkv():
    return [torch.randn(1, 2, 64, 64).to(torch.bfloat16) for _ in range(3)]


@pytest.mark.parametrize("which", [0, 1, 2])
@pytest.mark.parametrize("grad", [False, True])
def test_a_dual_tensor_is_refused(which, grad):
    x = _qkv()
    with fwAD.dual_level():
        x[which] = fwAD.make_dual(x[which], torch.ones_like(x[which]))
        with torch.set_grad_enabled(grad), pytest.raises(NotImplementedError):
            sage_attention(*x)


def test_transforms_of_torch_func_are_refused():
    q, k, v = _qkv()
    # (torch's own refusal of a torch.autograd.Function without rules is a RuntimeError, which NotImplementedError is too)
    with pytest.raises(RuntimeError):
        torch.func.jvp(lambda a: sage_attention(a, k, v), (q,), (torch.ones_like(q),))
    with pytest.raises(RuntimeError):
        torch.func.grad(lambda a: sage_attention(q, a, v).float().sum())(k)
    with pytest.raises(RuntimeError):
        torch.vmap(lambda a: sage_attention(q, k, a))(torch.stack([v, v]))


def test_plain_tensors_meet_the_tensor_checks():
    with pytest.raises(ValueError):       # on the CPU
        sage_attention(*_qkv())
