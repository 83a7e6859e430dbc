"""fp32 forward: values at masked positions stay out of the rows that do not attend them, and the logsumexp of large scores."""
import numpy as np
import pytest
import torch

from paper_2306_01160_amd import binding as sc
from paper_2306_01160_amd import pipeline

pytestmark = pytest.mark.gpu


def _labels(rng, variant, B, H, T, nb):
    if variant == "hash":
        return tuple(torch.from_numpy(rng.integers(0, nb, (B, H, T), dtype=np.int32)).cuda() for _ in range(2))
    return tuple(torch.from_numpy((rng.random((B, H, T)) < 0.7).astype(np.uint8)).cuda() for _ in range(2))


def _forward(variant, q, k, v, lq, lk, nb, strict, whole):
    if whole:
        if variant == "hash":
            return pipeline.hash_forward(q, k, v, lq, lk, nb, 0.125, need_bwd=False, strict=strict)[:2]
        return pipeline.qkdrop_forward(q, k, v, lq, lk, 0.125, need_bwd=False, strict=strict)[:2]
    B, H, T, d = q.shape
    seg = lambda x: x.reshape(B * H, *x.shape[2:])  # noqa: E731
    flags = sc.SCFA_FLAG_STRICT_CAUSAL if strict else 0
    tiles = sc.scfa_tile_config(d, sc.SCFA_F32)
    if variant == "hash":
        (qi, _, qo, qk), (ki, _, ko, kk) = sc.scfa_sort_by_bucket_pair(seg(lq), seg(lk), nb, want_sorted=False)
        rows = sc.scfa_gather_qkv(seg(q), seg(k), seg(v), qi, ki)
        work, _, _ = sc.scfa_block_ranges(sc.SCFA_HASH, qi, ki, qo, ko, nb, tiles, want_bwd=False, flags=flags)
        return sc.scfa_hash_attn_fwd(*rows, qk, kk, work, B, H, 0.125, flags=flags)
    (qi, nq), (ki, nk) = sc.scfa_compact_keep_pair(seg(lq), seg(lk))
    rows = sc.scfa_gather_qkv(seg(q), seg(k), seg(v), qi, ki, nq, nk)
    work, _, _ = sc.scfa_block_ranges(sc.SCFA_QKDROP, qi, ki, nq, nk, 1, tiles, want_bwd=False, flags=flags)
    return sc.scfa_qkdrop_attn_fwd(*rows, qi, ki, nq, work, B, H, 0.125, flags=flags)


@pytest.mark.parametrize("whole", [True, False])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("variant,T,nb,strict", [("hash", 200, 1, False), ("hash", 333, 20, True), ("hash", 700, 3, False),
                                                  ("qkdrop", 300, 1, False)])
def test_a_value_that_is_not_finite_reaches_only_the_rows_that_attend_it(variant, T, nb, strict, d, whole):
    """Later keys and, in items put together from short buckets, keys of other buckets share tiles with the rows they are masked
    for.  Bits: neither the scores nor the order of the sums depend on V."""
    rng = np.random.default_rng(T + d)
    B, H = 1, 2
    q, k, v = (torch.from_numpy(rng.standard_normal((B, H, T, d), dtype=np.float32)).cuda() for _ in range(3))
    lq, lk = _labels(rng, variant, B, H, T, nb)
    o, lse = (x.clone() for x in _forward(variant, q, k, v, lq, lk, nb, strict, whole))
    bad = {T - 3: ("nan", 5), T // 2: ("inf", 0), T // 2 + 1: ("-inf", d - 1), 7: ("inf", 33)}   # position -> value, column
    dirty = v.clone()
    for pos, (what, col) in bad.items():
        dirty[:, :, pos, col] = float(what)
    o2, lse2 = _forward(variant, q, k, dirty, lq, lk, nb, strict, whole)
    assert torch.equal(lse, lse2)
    at = torch.arange(T, device="cuda")
    reached = torch.zeros_like(o, dtype=torch.bool)
    for pos, (_, col) in bad.items():
        same = lq == lk[:, :, pos:pos + 1] if variant == "hash" else (lq != 0) & (lk[:, :, pos:pos + 1] != 0)
        reached[..., col] |= same & (at >= pos + int(strict))
    assert reached.any() and not torch.isfinite(o2[reached]).any()
    assert torch.equal(o[~reached], o2[~reached])


@pytest.mark.parametrize("d", [64, 128])
def test_logsumexp_keeps_the_bits_of_the_maximum(d):
    """Whole-number rows: scores and, at a scale of 1/8, their multiples are exact.  A row of one key has that score for its
    logsumexp, to the bit; with more keys the addition rounds once (half a unit in the last place) and the sum's logarithm
    carries the rounding of exp2, log2 and at most 200 additions, a few 2^-24 of a number of at most log 200."""
    rng = np.random.default_rng(d)
    T, tau = 200, 0.125
    q, k = (rng.integers(-12, 13, (1, 2, T, d)).astype(np.float32) for _ in range(2))
    v = rng.standard_normal((1, 2, T, d), dtype=np.float32)
    gq, gk, gv = (torch.from_numpy(x).cuda() for x in (q, k, v))
    own = torch.arange(T, dtype=torch.int32, device="cuda").expand(1, 2, T).contiguous()
    _, lse, _ = pipeline.hash_forward(gq, gk, gv, own, own, T, tau, need_bwd=False)
    assert np.array_equal(lse.cpu().numpy(), (np.einsum("bhtd,bhtd->bht", q, k) * tau).astype(np.float32))
    one = torch.zeros_like(own)
    _, lse, _ = pipeline.hash_forward(gq, gk, gv, one, one, 1, tau, need_bwd=False)
    s = np.einsum("bhid,bhjd->bhij", q.astype(np.float64), k.astype(np.float64)) * tau
    s = np.where(np.tril(np.ones((T, T), bool)), s, -np.inf)
    m = s.max(-1)
    want = m + np.log(np.exp(s - m[..., None]).sum(-1))
    assert np.all(np.abs(lse.cpu().numpy() - want) <= 0.5 * np.spacing(np.abs(want).astype(np.float32)) + 2.0 ** -20)
