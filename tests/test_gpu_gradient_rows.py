"""Gradients row by row: rows of dO of very different size, small values, small softmax scales.

Every gradient row is a sum; its error is held against the sum of its terms' magnitudes, so that no row hides behind another
one's size.  With P recomputed from a logsumexp that is off by up to 4e-4 (the forward's own figure), rounded to 11 bits (2^-11),
dP - D and their product rounded likewise, and D off by the rounding of O's fp16 copy (2^-12 |dO| |O|):
  dV_j   1e-3 of sum_i P_ij |dO_i|
  dK_j   2e-3 of tau sum_i P_ij (|dP_ij - D_i| + 2^-1 |dO_i| |O_i|) |q_i|, and 2^-24 of the largest |dO| of the segment times
         tau sum_i |q_i| over the rows that see j: dS is an fp16 number on one scale for the rows of a sum
  dQ_i   2e-3 of tau sum_j P_ij (|dP_ij - D_i| + 2^-1 |dO_i| |O_i|) |k_j|, and 2^-24 of the row's largest |dO| times tau sum_j |k_j|
(norms over the head dimension)."""
import numpy as np
import pytest
import torch

from paper_2306_01160_amd import binding as sc
from paper_2306_01160_amd import workloads as W

from gpu_util import labels, run_gpu, seg64

pytestmark = pytest.mark.gpu


def _reference(wl):
    """fp64: gradients and the sums of the magnitudes of their terms"""
    lq, lk = labels(wl)
    Q, K, V, dO = (seg64(wl, a) for a in (wl.q, wl.k, wl.v, wl.do))
    at = np.arange(wl.T)
    grads, bounds = [], []
    norm = lambda x: np.linalg.norm(x, axis=-1)  # noqa: E731
    for s in range(wl.S):
        allowed = (lq[s][:, None] == lk[s][None, :]) & (at[None, :] <= at[:, None])
        x = np.where(allowed, wl.tau * (Q[s] @ K[s].T), -np.inf)
        m = x.max(-1, keepdims=True)
        P = np.exp(x - np.where(np.isfinite(m), m, 0.0))
        total = P.sum(-1, keepdims=True)
        P /= np.where(total > 0, total, 1.0)
        O = P @ V[s]
        dP = dO[s] @ V[s].T
        D = (dO[s] * O).sum(-1, keepdims=True)
        dS = P * (dP - D)
        grads.append((wl.tau * dS @ K[s], wl.tau * dS.T @ Q[s], P.T @ dO[s]))
        size = np.abs(dS) + 0.5 * P * (norm(dO[s]) * norm(O))[:, None]
        rowmax = np.abs(dO[s]).max(-1)
        bounds.append((wl.tau * (2e-3 * size @ norm(K[s]) + 2.0 ** -24 * rowmax * (allowed @ norm(K[s]))),
                       wl.tau * (2e-3 * size.T @ norm(Q[s]) + 2.0 ** -24 * rowmax.max() * (allowed.T @ norm(Q[s]))),
                       1e-3 * P.T @ norm(dO[s])))
    return grads, bounds


def _check(wl):
    _, _, got, _ = run_gpu(wl)
    grads, bounds = _reference(wl)
    for i, name in enumerate(("dQ", "dK", "dV")):
        g = got[i].cpu().numpy().reshape(wl.S, wl.T, wl.d).astype(np.float64)
        assert np.isfinite(g).all(), name
        for s in range(wl.S):
            err = np.linalg.norm(g[s] - grads[s][i], axis=-1)
            over = err / np.maximum(bounds[s][i], 1e-300)
            assert (over <= 1.0).all(), (name, s, int(over.argmax()), float(over.max()))


def _scale_rows(wl, power):
    wl.do = W.round_to_bf16(wl.do * np.exp2(np.asarray(power, np.float64)).astype(np.float32).reshape(1, 1, -1, 1))
    return wl


def _flat(T, d, nb, seed, B=1, H=1):
    wl = W.hash_uniform(seed, B, H, T, d, nb)
    wl.q = W.round_to_bf16(wl.q * np.float32(0.25))          # flat rows: probabilities down to nb / T
    return wl


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("v_power", [0, -9, -12, -13, 9])
@pytest.mark.parametrize("gap", [0, 3, 10, 14])
@pytest.mark.parametrize("nb", [1, 2])
def test_one_large_row_before_small_ones(nb, gap, v_power, d):
    """All keys but the first are seen by small rows only, and share an item with the row that sets the scale.  (One bucket of 1500 at
    d = 64: two groups of wavefronts share the item's tiles.)"""
    wl = _flat(1500, d, nb, 11 + gap)
    wl.v = np.ldexp(wl.v, v_power)
    _check(_scale_rows(wl, np.where(np.arange(wl.T) == 0, 0, -gap)))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("gap,v_power", [(14, 0), (10, 9), (2, 0)])
def test_launches_of_their_own(gap, v_power, d):
    """Under the event timers the dK/dV and the dQ items have a launch each; same bits, wide ranges of dO or not."""
    wl = _flat(1100, d, 3, 31)
    wl.v = np.ldexp(wl.v, v_power)
    wl = _scale_rows(wl, np.where(np.arange(wl.T) % 150 == 0, 0, -gap))
    _, _, together, _ = run_gpu(wl)
    sc.scfa_prof_reset()
    sc.scfa_prof_enable(True)
    try:
        _, _, apart, _ = run_gpu(wl)
        assert sc.scfa_prof_read("bwd_dkdv")[1] == 1 and sc.scfa_prof_read("bwd_dq")[1] == 1
    finally:
        sc.scfa_prof_enable(False)
        sc.scfa_prof_reset()
    for name, a, b in zip(("dQ", "dK", "dV"), together, apart):
        assert torch.equal(a, b), name
    _check(wl)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("v_power", [0, -9, -13])
@pytest.mark.parametrize("spread", [1, 2, 4])
def test_rows_of_random_size(spread, v_power, d):
    wl = _flat(2048, d, 1, 5 + spread)
    wl.v = np.ldexp(wl.v, v_power)
    _check(_scale_rows(wl, np.clip(np.rint(spread * np.random.default_rng(spread).standard_normal(wl.T)), -10, 4)))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("T,nb,B,H", [(900, 40, 1, 3), (700, 5, 2, 2), (1100, 2, 4, 48)])
def test_buckets_of_different_size_share_a_scale(T, nb, B, H, d):
    """Short buckets are put together in items, and the entries that the scale is read from cover rows of several buckets."""
    wl = W.hash_uniform(17, B, H, T, d, nb)
    size = -2.0 * (wl.lab_q % 7)
    wl.do = W.round_to_bf16(wl.do * np.exp2(size).astype(np.float32)[..., None])
    if B * H > 4:                                            # the CPU's share
        keep = slice(0, 1)
        small = W.hash_uniform(17, 1, 1, T, d, nb)
        for a in ("q", "k", "v", "do", "lab_q", "lab_k"):
            setattr(small, a, np.ascontiguousarray(getattr(wl, a)[keep, :1]))
        _, _, all_rows, _ = run_gpu(wl)
        _, _, one, _ = run_gpu(small)
        grads, bounds = _reference(small)
        for i, name in enumerate(("dQ", "dK", "dV")):
            for g in (all_rows[i][:1, :1], one[i]):
                err = np.linalg.norm(g.cpu().numpy().reshape(T, d) - grads[0][i], axis=-1)
                assert (err <= bounds[0][i]).all(), (name, float((err / bounds[0][i]).max()))
        return
    _check(wl)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("v_power,gap", [(7, 0), (7, 12), (11, 12)])
def test_large_values_against_small_rows(gap, v_power, d):
    """A common offset of the values makes |D| large: with 2^11 and 64 or 128 elements it passes 65504 once a row of dO is brought to
    [1, 2).  The rows that set the scale of the segment have one large element and a small D themselves."""
    wl = _flat(600, d, 2, 23)
    wl.v = W.round_to_bf16(np.ldexp(np.abs(wl.v) + np.float32(1.0), v_power))
    wl.do = np.abs(wl.do)
    wl.do[:, :, :4] *= np.float32(2.0 ** -6)
    wl.do[:, :, :4, 0] = 1.0
    _check(_scale_rows(wl, np.where(np.arange(wl.T) < 4, 0, -gap)))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("tau,rows", [(4e-5, "zero"), (1e-5, "zero"), (8e-6, "small"), (4e-5, "tiny"), (0.125, "tiny")])
def test_small_scales(tau, rows, d):
    """Rows of zeros (padding) and small rows under a small softmax scale: the row's power of two is no part of what limits
    |LSE| / tau, and a row of zeros has none."""
    wl = W.hash_uniform(29, 1, 2, 700, d, 3)
    wl.__class__ = type("Scaled", (W.Workload,), {"tau": tau})
    power = {"zero": 0.0, "small": -27.0, "tiny": -100.0}[rows]
    wl = _scale_rows(wl, np.full(wl.T, power))
    wl.do[:, :, ::5] = 0.0
    wl.do[:, :, 600:] = 0.0
    _check(wl)
