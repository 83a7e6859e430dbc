"""The order in which one launch takes the items of the two gradients, and dQ items that it leaves to the next: every item is done once, so
the gradients have the bits that a launch for each kind gives (which the event timers ask for), dropped rows zero.  Segments of one call
that keep more queries than keys, more keys than queries, all, none; fewer than 8 segments and more; both head dimensions; calls beyond the
sizes at which some segments' dQ items are left, among segments whose are not; hash buckets short and long, items shared by two groups."""
import pytest
import torch

from paper_2306_01160_amd import binding as sc
from paper_2306_01160_amd import pipeline

pytestmark = pytest.mark.gpu

MIXED = [(1.0, 1.0), (0.5, 0.5), (0.9, 0.2), (0.2, 0.9), (0.0, 1.0), (1.0, 0.0), (0.3, 0.28)]


def _check(forward, backward, launches):
    _, _, ctx = forward()
    plain = backward(ctx)
    sc.scfa_prof_reset()
    sc.scfa_prof_enable(True)
    try:
        timed = backward(ctx)
        assert sc.scfa_prof_read("bwd_dkdv")[1] == launches and sc.scfa_prof_read("bwd_dq")[1] == launches
    finally:
        sc.scfa_prof_enable(False)
        sc.scfa_prof_reset()
    for name, a, b in zip(("dQ", "dK", "dV"), plain, timed):
        assert torch.isfinite(a).all() and torch.equal(a, b), name
    return plain


def _rows(S, T, d):
    gen = torch.Generator(device="cuda"); gen.manual_seed(S * T)
    return gen, [torch.randn((1, S, T, d), device="cuda", generator=gen).bfloat16() for _ in range(4)]


@pytest.mark.parametrize("S,T,d", [(7, 1500, 64), (7, 1500, 128), (3, 9000, 64), (16, 3000, 64), (9, 2000, 128), (40, 3000, 64), (20, 3000, 128),
                                   (7, 11500, 128), (2, 40000, 128), (4, 56000, 64)])
def test_dropping(S, T, d):
    gen, (q, k, v, do) = _rows(S, T, d)
    keep = torch.tensor([MIXED[s % len(MIXED)] for s in range(S)], device="cuda").T.reshape(2, 1, S, 1)
    kq, kk = (torch.rand((2, 1, S, T), device="cuda", generator=gen) < keep).to(torch.uint8)
    grads = _check(lambda: pipeline.qkdrop_forward(q, k, v, kq, kk, 0.125), lambda ctx: pipeline.qkdrop_backward(ctx, do), 1)
    for g, kept in zip(grads, (kq, kk, kk)):
        assert not g[kept == 0].any()


@pytest.mark.parametrize("S,T,d,nb", [(4, 2816, 128, 34), (12, 1000, 128, 16), (3, 9000, 128, 4), (1, 5000, 128, 6), (6, 4096, 64, 8), (13, 3000, 64, 20),
                                      (12, 2560, 64, 2)])
def test_hash(S, T, d, nb):
    gen, (q, k, v, do) = _rows(S, T, d)
    bq, bk = (torch.randint(0, nb, (1, S, T), device="cuda", generator=gen, dtype=torch.int32) for _ in range(2))
    _check(lambda: pipeline.hash_forward(q, k, v, bq, bk, nb, 0.125), lambda ctx: pipeline.hash_backward(ctx, do), 1)
