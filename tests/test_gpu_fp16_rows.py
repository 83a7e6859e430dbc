"""Whole passes on rows that are in the fp16 compute format already, against the single entry points: same launches, same
bits.  Both sides of the sizes that sort, list and gather in one launch, and both head dimensions."""
import pytest
import torch

from paper_2306_01160_amd import binding as sc
from paper_2306_01160_amd import pipeline

pytestmark = pytest.mark.gpu


def _equal(pairs):
    for name, a, b in pairs:
        assert torch.equal(a, b), name


@pytest.mark.parametrize("T", [1, 513, 4096, 4097, 9001])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("variant", ["hash", "qkdrop"])
def test_fp16_rows(variant, T, d):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(T + d)
    B, H, nb = 1, 3, 5
    S = B * H
    # fp16 numbers that are bf16 numbers too: the bf16 pass has the same products
    q, k, v = (torch.randn((B, H, T, d), device="cuda", generator=gen).to(torch.bfloat16) for _ in range(3))
    do = torch.randn((B, H, T, d), device="cuda", generator=gen).to(torch.bfloat16)
    rows = [torch.where(x.abs() < 2.0 ** -9, torch.zeros_like(x), x) for x in (q, k, v)]
    h = [x.to(torch.float16) for x in rows]
    seg = lambda x: x.reshape(S, *x.shape[2:])  # noqa: E731
    if variant == "hash":
        lq, lk = (torch.randint(0, nb, (B, H, T), device="cuda", generator=gen, dtype=torch.int32) for _ in range(2))
        o, lse, ctx = pipeline.hash_forward(*h, lq, lk, nb, 0.125)
        o2, lse2, _ = pipeline.hash_forward(*rows, lq, lk, nb, 0.125)
        got = pipeline.hash_backward(ctx, do)
        (qi, _, qo, qk), (ki, _, ko, kk) = sc.scfa_sort_by_bucket_pair(seg(lq), seg(lk), nb, want_sorted=False)
        perm = sc.scfa_gather_qkv(*(seg(x) for x in h), qi, ki)
        fw, bw, _ = sc.scfa_block_ranges(sc.SCFA_HASH, qi, ki, qo, ko, nb, sc.scfa_tile_config(d, sc.SCFA_BF16))
        o1, lse1 = sc.scfa_hash_attn_fwd(*perm, qk, kk, fw, B, H, 0.125)
        want = sc.scfa_hash_attn_bwd(*perm, qk, kk, fw, bw, o1, lse1, do, B, H, 0.125)
        o3, lse3, _ = pipeline.hash_forward(*h, lq, lk, nb, 0.125, need_bwd=False)
    else:
        lq, lk = ((torch.rand((B, H, T), device="cuda", generator=gen) < 0.6).to(torch.uint8) for _ in range(2))
        o, lse, ctx = pipeline.qkdrop_forward(*h, lq, lk, 0.125)
        o2, lse2, _ = pipeline.qkdrop_forward(*rows, lq, lk, 0.125)
        got = pipeline.qkdrop_backward(ctx, do)
        (qi, nq), (ki, nk) = sc.scfa_compact_keep_pair(seg(lq), seg(lk))
        perm = sc.scfa_gather_qkv(*(seg(x) for x in h), qi, ki, nq, nk)
        fw, bw, _ = sc.scfa_block_ranges(sc.SCFA_QKDROP, qi, ki, nq, nk, 1, sc.scfa_tile_config(d, sc.SCFA_BF16))
        o1, lse1 = sc.scfa_qkdrop_attn_fwd(*perm, qi, ki, nq, fw, B, H, 0.125)
        want = sc.scfa_qkdrop_attn_bwd(*perm, qi, ki, nq, nk, fw, bw, o1, lse1, do, B, H, 0.125)
        o3, lse3, _ = pipeline.qkdrop_forward(*h, lq, lk, 0.125, need_bwd=False)
    assert o.dtype == torch.bfloat16 and ctx.o_f16 is None
    _equal([("O", o, o1), ("LSE", lse, lse1), ("O of bf16 rows", o, o2), ("LSE of bf16 rows", lse, lse2),
            ("O without backward", o, o3), ("LSE without backward", lse, lse3)])
    _equal(zip(("dQ", "dK", "dV"), got, want))
