"""Gradient rows leave a workgroup through LDS, whole rows at a time: last items of one row, of a row less and more than a wavefront's
32, of a whole tile; both head dimensions, one group of wavefronts an item and two; tolerances as in test_gpu_attention_parity.py."""
import pytest
import torch

from gpu_util import assert_within, compare_backward, run_gpu
from paper_2306_01160_amd import pipeline
from paper_2306_01160_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [1, 31, 32, 33, 97, 128, 129, 1024 + 65])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("strict", [False, True])
def test_one_bucket(T, d, strict):
    wl = W.hash_uniform(6100 + T, 1, 2, T, d, 1)
    wl.meta["strict"] = strict
    assert_within(compare_backward(wl, run_gpu(wl)[2]), wl.dtype)


@pytest.mark.parametrize("T,pq,pk,d", [(129, 0.01, 0.9, 64), (700, 0.05, 0.03, 128), (2304, 0.5, 0.9, 64)])
def test_dropped_rows_are_zero(T, pq, pk, d):
    wl = W.qkdrop_bernoulli(6200 + T, 1, 2, T, d, pq, pk)
    dq, dk, dv = run_gpu(wl)[2]
    assert_within(compare_backward(wl, (dq, dk, dv)), wl.dtype)
    for g, keep in ((dq, wl.lab_q), (dk, wl.lab_k), (dv, wl.lab_k)):
        assert not g.cpu().numpy()[keep == 0].any()


@pytest.mark.parametrize("S,T,d", [(28, 8193, 64), (15, 8191, 128)])
def test_large_steps_have_the_bits_of_their_parts(S, T, d):
    """Beyond 256 MB of rows the pre-pass reads past the caches; a part of the segments stays below."""
    gen = torch.Generator(device="cuda"); gen.manual_seed(T)
    q, k, v, do = (torch.randn((S, 1, T, d), device="cuda", generator=gen).bfloat16() for _ in range(4))
    bq, bk = (torch.randint(0, 16, (S, 1, T), device="cuda", generator=gen, dtype=torch.int32) for _ in range(2))
    def step(i0, i1):
        q_, k_, v_, do_, bq_, bk_ = (x[i0:i1] for x in (q, k, v, do, bq, bk))
        o, lse, ctx = pipeline.hash_forward(q_, k_, v_, bq_, bk_, 16, 0.125)
        return (o, lse) + tuple(pipeline.hash_backward(ctx, do_))
    parts = [step(0, 6), step(6, S)]
    for name, whole, a, b in zip(("O", "LSE", "dQ", "dK", "dV"), step(0, S), *parts):
        assert torch.equal(whole, torch.cat([a, b])), name
