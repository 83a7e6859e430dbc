"""fp32 forward at d = 64: numbers whose products or pieces leave what bf16 pieces can carry come out as from fp32 products."""
import math

import pytest
import torch

from paper_2306_01160_amd import pipeline

pytestmark = pytest.mark.gpu

TAU, FLT_MAX = 0.125, torch.finfo(torch.float32).max


def _reference(q, k, v, allowed):
    """softmax(TAU q k^T) v over allowed pairs in fp64; scores below fp32's range take no part"""
    s = torch.matmul(q.double(), k.double().transpose(-1, -2).contiguous())
    s = s.masked_fill(~allowed | (s < -FLT_MAX), -float("inf")) * TAU
    lse = torch.logsumexp(s, -1)
    p = torch.where(torch.isneginf(s), 0.0, torch.exp(s - lse.clamp(min=-1e300)[..., None]))
    return torch.matmul(p, v.double()), lse


def _inputs(T, nb):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(T + nb)
    q, k, v = (torch.randn((1, 2, T, 64), device="cuda", generator=gen) for _ in range(3))
    lq, lk = (torch.randint(0, nb, (1, 2, T), device="cuda", generator=gen, dtype=torch.int32) for _ in range(2))
    lq[..., 0] = lk[..., 0] = 0                # the first row takes the first key
    return q, k, v, lq, lk


def _allowed(lq, lk):
    at = torch.arange(lq.shape[-1], device="cuda")
    return (lq[..., :, None] == lk[..., None, :]) & (at[:, None] >= at[None, :])


# a forward for a backward sorts in a launch of its own; the other shares its launch with the attention at these sizes
@pytest.mark.parametrize("need_bwd", [False, True])
@pytest.mark.parametrize("pos", [0, 40])
@pytest.mark.parametrize("q5,k5", [(2005.0, -3e38), (1.004, 3.385e38), (1.004, -3.385e38)])
def test_finite_numbers_whose_score_ends_the_range(q5, k5, pos, need_bwd):
    """One score beyond fp32's range, or so near its end that the product of the leading pieces is beyond it."""
    nb = 2
    q, k, v, lq, lk = _inputs(300, nb)
    lk[..., pos] = 0
    q[..., 5] = q5
    k[..., 5] = 0.0
    k[:, :, pos, 5] = k5
    o, lse, _ = pipeline.hash_forward(q, k, v, lq, lk, nb, TAU, need_bwd=need_bwd)
    o_ref, lse_ref = _reference(q, k, v, _allowed(lq, lk))
    some = torch.isfinite(lse_ref)
    assert torch.equal(torch.isfinite(lse), some) and torch.isfinite(o).all()
    assert float((o - o_ref).abs().max()) < 5e-6
    assert float(((lse - lse_ref)[some].abs() / lse_ref[some].abs().clamp(min=1.0)).max()) < 1e-5
