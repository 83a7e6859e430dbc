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
