"""The gather reads rows through the caches up to a size and past them above (beyond 4096 tokens, where it is a launch of its own):
a forward of one segment more than the limit has the bits of one without its first or its last, which lie below, and a gather the rows it is told to fetch."""
import pytest
import torch

from paper_2306_01160_amd import binding as sc
from paper_2306_01160_amd import pipeline

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d", [(4999, 64), (4099, 128)])
@pytest.mark.parametrize("drop", [False, True])
@pytest.mark.parametrize("train", [False, True])
def test_forward_on_both_sides_of_the_limit(T, d, drop, train):
    S = ((11 if train else 16) * (2 if drop else 1) << 20) // (T * d * 2) + 1
    gen = torch.Generator(device="cuda"); gen.manual_seed(T)
    q, k, v = (torch.randn((1, S, T, d), device="cuda", generator=gen).bfloat16() for _ in range(3))
    lq, lk = (torch.randint(0, 2 if drop else 9, (1, S, T), device="cuda", generator=gen, dtype=torch.int32) for _ in range(2))
    if drop:
        lq, lk = lq.to(torch.uint8), lk.to(torch.uint8)
    def forward(i0, i1):
        part = [x[:, i0:i1] for x in (q, k, v, lq, lk)]
        return (pipeline.qkdrop_forward(*part, 0.125, need_bwd=train) if drop else pipeline.hash_forward(*part, 9, 0.125, need_bwd=train))[:2]
    whole = forward(0, S)
    for i0, i1 in ((0, S - 1), (1, S)):
        for name, x, part in zip(("O", "LSE"), whole, forward(i0, i1)):
            assert torch.equal(x[:, i0:i1], part), name


@pytest.mark.parametrize("over", [False, True])
def test_gathered_rows(over):
    T, d = 1003, 64
    S = (16 << 20) // (T * d * 2) + over
    gen = torch.Generator(device="cuda"); gen.manual_seed(S)
    x = torch.randn((S, T, d), device="cuda", generator=gen).bfloat16()
    idx = torch.stack([torch.randperm(T, device="cuda", generator=gen) for _ in range(S)]).to(torch.int32)
    want = torch.gather(x, 1, idx.long()[..., None].expand(-1, -1, d))
    assert torch.equal(sc.scfa_gather_rows(x, idx, out=torch.empty_like(x)), want)
