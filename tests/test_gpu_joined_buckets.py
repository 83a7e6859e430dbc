"""Consecutive buckets that share a work item, up to two tiles of rows on the ranged side where there are many rows: the schedule's own
rules (those of test_gpu_integer_passes.py), and the attention over such items against the oracle; few buckets and more than 64, some
without queries or keys, both mask forms; tolerances as in test_gpu_attention_parity.py."""
import numpy as np
import pytest

from gpu_util import assert_within, compare_backward, compare_forward, run_gpu
from paper_2306_01160_amd import binding as sc
from paper_2306_01160_amd import workloads as W
from test_gpu_integer_passes import _check_schedule

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,T,nb", [(129, 1024, 16), (65, 2050, 31), (33, 4100, 130)])
@pytest.mark.parametrize("strict", [False, True])
def test_schedule(S, T, nb, strict):
    rng = np.random.default_rng(T + nb)
    bq, bk = (rng.integers(0, nb, (S, T)).astype(np.int32) for _ in range(2))
    bk[bk == 2] = 0          # a bucket without keys
    bq[bq == 1] = 0          # and one without queries
    merged = _check_schedule(sc.SCFA_HASH, bq, bk, nb, sc.scfa_tile_config(64, sc.SCFA_BF16), strict=strict)
    assert merged > S * nb // 4


@pytest.mark.parametrize("T,d,nb", [(1025, 64, 16), (1024, 128, 13)])
@pytest.mark.parametrize("strict", [False, True])
def test_attention(T, d, nb, strict):
    wl = W.hash_uniform(7600 + T, 1, 130, T, d, nb)
    wl.meta["strict"] = strict
    o, lse, grads, _ = run_gpu(wl)
    segs = [0, 1, 129]
    assert_within(compare_forward(wl, o, lse, segs=segs), wl.dtype)
    assert_within(compare_backward(wl, grads, segs=segs), wl.dtype)
