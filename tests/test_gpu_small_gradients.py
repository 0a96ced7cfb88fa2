"""Gradients far from 1: dQ, dK and dV of dO times a power of two are theirs times it."""
import pytest
import torch

from paper_2603_02170_amd import binding

pytestmark = pytest.mark.gpu


# Every step is linear in dO, and its rounding scales with it while FP32's normal range is not left.  At 2^-102 the scales' products (about 2^-123) and the sums are
# inside; what is not, products of the smallest probabilities, is below 2^-20 of the sums, which moves a bf16 result by its last place (2^-8) in 1e-3 of the
# values: 1e-4 in norm.  At 2^-110 dQ alone: dK's and dV's scales leave the range there.  An emulation of dQ's sums in FP32 gives 1e-6 with half of the 2^26 in
# the weights (kDqWeight) and 1.3e-3 with all of it made up at the end; at 2^-102 4e-9 and 6e-5, which the bound would not tell apart.
# 8 heads take the form of dQ with one Q block per workgroup, 200 the one with two (use_dq_split).
@pytest.mark.parametrize("exponent", [-110, -102, -60, 60])
@pytest.mark.parametrize("heads,N,d", [(8, 300, 128), (8, 300, 64), (200, 300, 128), (200, 300, 64)])
def test_gradients_scale_with_dO(heads, N, d, exponent):
    g = torch.Generator(device="cuda").manual_seed(heads + d)
    Q, K, V, dO = (torch.randn((1, heads, N, d), generator=g, device="cuda").to(torch.bfloat16) for _ in range(4))
    p = binding.SageParams(1, heads, N, d, causal=True)
    O, L = binding.sagebwd_fwd(Q, K, V, p)
    want = binding.sagebwd_bwd(Q, K, V, O, dO, L, p)
    got = binding.sagebwd_bwd(Q, K, V, O, (dO.double() * 2.0 ** exponent).to(torch.bfloat16), L, p)
    torch.cuda.synchronize()
    names = ("dQ",) if exponent < -102 else ("dQ", "dK", "dV")
    for name, a, b in zip(names, got, want):
        a, b = a.double() * 2.0 ** -exponent, b.double()
        assert b.abs().max() > 0.05, name
        assert (a - b).norm() <= 1e-4 * b.norm(), (name, float((a - b).norm() / b.norm()))
