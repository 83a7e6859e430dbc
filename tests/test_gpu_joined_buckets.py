"""Consecutive buckets that share a work item: the schedule's own rules (those of test_gpu_integer_passes.py), the attention over such
items against the oracle (few buckets and more than 64, some without queries or keys, both mask forms), and that only buckets shorter
than a tile on both sides share one, however many rows a call has, so that a bucket's values do not reach others; tolerances as in
test_gpu_attention_parity.py."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import assert_within, compare_backward, compare_forward, labels, run_gpu, seg64
from paper_2306_01160_amd import binding as sc
from paper_2306_01160_amd import workloads as W
from test_gpu_integer_passes import _check_schedule

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,T,nb", [(129, 1024, 24), (65, 2050, 64), (33, 4100, 130)])
@pytest.mark.parametrize("strict", [False, True])
def test_schedule(S, T, nb, strict):
    rng = np.random.default_rng(T + nb)
    bq, bk = (rng.integers(0, nb, (S, T)).astype(np.int32) for _ in range(2))
    bk[bk == 2] = 0          # a bucket without keys
    bq[bq == 1] = 0          # and one without queries
    merged = _check_schedule(sc.SCFA_HASH, bq, bk, nb, sc.scfa_tile_config(64, sc.SCFA_BF16), strict=strict)
    assert merged > S * nb // 4


@pytest.mark.parametrize("T,d,nb", [(1025, 64, 26), (1024, 128, 24)])
@pytest.mark.parametrize("strict", [False, True])
def test_attention(T, d, nb, strict):
    wl = W.hash_uniform(7600 + T, 1, 130, T, d, nb)
    wl.lab_k[wl.lab_k == 2] = 0
    wl.lab_q[wl.lab_q == 1] = 0
    wl.meta["strict"] = strict
    o, lse, grads, ctx = run_gpu(wl)
    segs = [0, 1, 129]
    assert (ctx.fwd_work[segs][..., 6] > 1).any(1).all() and (ctx.bwd_work[segs][..., 6] > 1).any(1).all()
    assert_within(compare_forward(wl, o, lse, segs=segs), wl.dtype)
    assert_within(compare_backward(wl, grads, segs=segs), wl.dtype)


def _labels(rng, S, sizes):
    """Bucket b has sizes[b] rows of every segment."""
    return np.stack([rng.permutation(np.repeat(np.arange(len(sizes), dtype=np.int32), sizes)) for _ in range(S)])


@pytest.mark.parametrize("S,q_sizes,k_sizes", [(130, [64] * 16, [70, 58] * 8), (130, [100] * 10 + [24], [24] * 10 + [784]),
                                               (20, [16] * 129 + [6192], [64] * 129), (20, [64] * 129, [16] * 129 + [6192])])
def test_a_tile_of_rows_keeps_a_bucket_apart(S, q_sizes, k_sizes):
    rng = np.random.default_rng(S)
    nb = max(len(q_sizes), len(k_sizes))
    q_sizes, k_sizes = (np.array(x + [0] * (nb - len(x))) for x in (q_sizes, k_sizes))
    fm, fn, bn, bm = sc.scfa_tile_config(64, sc.SCFA_BF16)
    lab_q, lab_k = (torch.from_numpy(_labels(rng, S, x)).cuda() for x in (q_sizes, k_sizes))
    q_idx, _, q_off = sc.scfa_sort_by_bucket(lab_q, nb)
    k_idx, _, k_off = sc.scfa_sort_by_bucket(lab_k, nb)
    fwd, bwd, _ = sc.scfa_block_ranges(sc.SCFA_HASH, q_idx, k_idx, q_off, k_off, nb, (fm, fn, bn, bm))
    close = 0                # buckets that would join under a limit of two tiles
    for work, tiled, ranged, tile in ((fwd, q_sizes, k_sizes, fn), (bwd, k_sizes, q_sizes, bm)):
        close += ((ranged >= tile) & (ranged < 2 * tile) & (tiled <= 64)).sum()
        for bucket, n in work[..., 5:7].reshape(-1, 2).cpu().numpy():
            assert n <= 1 or (ranged[bucket:bucket + n] < tile).all(), (bucket, n)
    assert close >= 10


def _part(wl, i0, i1):
    part = W.Workload(**{**wl.__dict__, "H": i1 - i0})
    for name in ("q", "k", "v", "do", "lab_q", "lab_k"):
        setattr(part, name, getattr(wl, name)[:, i0:i1])
    return part


def _same(a, b):
    return bool(((a == b) | ((a != a) & (b != b))).all())


@pytest.mark.parametrize("d", [64, 128])
def test_a_value_that_is_not_finite_stays_in_its_bucket(d):
    S, T, nb = 130, 1024, 16
    wl = W.hash_uniform(7700, 1, S, T, d, nb)
    rng = np.random.default_rng(d)
    wl.lab_q[0], wl.lab_k[0] = _labels(rng, S, [64] * nb), _labels(rng, S, [64] * nb)
    first = (wl.lab_k[0] == 3).argmax(1)              # the first key of bucket 3, of two kinds
    wl.v[0, np.arange(S), first, 0] = np.where(np.arange(S) % 2 == 0, np.inf, np.nan)
    o, lse, grads, _ = run_gpu(wl)
    out = torch.from_numpy(wl.lab_q != 3).cuda()
    assert torch.isfinite(o[out]).all() and not torch.isnan(lse[out]).any()
    assert not torch.isfinite(o[~out]).all()
    parts = [run_gpu(_part(wl, a, b)) for a, b in ((0, 60), (60, S))]
    for name, whole, a, b in zip(("O", "LSE", "dQ", "dK", "dV"), (o, lse) + tuple(grads), *((p[0], p[1]) + tuple(p[2]) for p in parts)):
        assert _same(whole, torch.cat([a, b], 1)), name


@pytest.mark.parametrize("d", [64, 128])
def test_a_bucket_keeps_its_own_scale_of_dO(d):
    """Buckets of 96 queries and 24 keys, four whole blocks of dO rows (three of 128) 2^18 below the next four: each row of dV to
    1e-3 of the sum of its terms' magnitudes, as in test_gpu_gradient_rows.py."""
    S, nb = 130, 11
    q_sizes, k_sizes = [96] * 10 + [64], [24] * 10 + [784]
    wl = W.hash_uniform(7800, 1, S, 1024, d, nb)
    rng = np.random.default_rng(d)
    wl.lab_q[0], wl.lab_k[0] = _labels(rng, S, q_sizes), _labels(rng, S, k_sizes)
    wl.do[...] = wl.do * np.where(wl.lab_q < 4, np.float32(2.0 ** -18), np.float32(1.0))[..., None]
    o, lse, grads, _ = run_gpu(wl)
    parts = [run_gpu(_part(wl, a, b)) for a, b in ((0, 60), (60, S))]
    for name, whole, a, b in zip(("O", "LSE", "dQ", "dK", "dV"), (o, lse) + tuple(grads), *((p[0], p[1]) + tuple(p[2]) for p in parts)):
        assert _same(whole, torch.cat([a, b], 1)), name
    lq, lk = labels(wl)
    Q, K, V, dO = (seg64(wl, a)[:1] for a in (wl.q, wl.k, wl.v, wl.do))
    want = oracle.attention_backward(Q, K, V, dO, lq[:1], lk[:1], oracle.HASH, wl.tau)[2][0]
    x = np.where((lq[0][:, None] == lk[0][None]) & (np.arange(1024)[None] <= np.arange(1024)[:, None]), wl.tau * Q[0] @ K[0].T, -np.inf)
    P = np.exp(x - np.where(np.isfinite(x.max(1)), x.max(1), 0.0)[:, None])
    P /= np.maximum(P.sum(1, keepdims=True), 1e-300)
    err = np.linalg.norm(grads[2][0, 0].cpu().numpy() - want, axis=1)
    assert (err <= 1e-3 * (P.T @ np.linalg.norm(dO[0], axis=1)) + 1e-30).all()
