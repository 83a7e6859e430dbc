"""Gradient rows leave a workgroup through LDS, whole rows at a time: last items of one row, of a row less and more than a wavefront's
32, of a whole tile; both head dimensions, one group of wavefronts an item and two; tolerances as in test_gpu_attention_parity.py."""
import pytest

from gpu_util import assert_within, compare_backward, run_gpu
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
