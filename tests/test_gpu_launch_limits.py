"""Launches of more threads than one grid takes (2^32): many segments times many buckets, most items empty."""
import pytest
import torch

from paper_2306_01160_amd import pipeline

pytestmark = pytest.mark.gpu


def _inputs(S, T, d, nb, dtype):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(S)
    rows = [torch.randn((S, 1, T, d), device="cuda", generator=gen).to(dtype) for _ in range(4)]
    bucket = torch.randint(0, nb, (S, 1, T), device="cuda", generator=gen, dtype=torch.int32)
    return rows, bucket


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_forward_beyond_one_grid(dtype):
    S, T, d, nb = 65535, 2, 64, 256              # 65535 x 257 items of 256 threads
    (q, k, v, _), bucket = _inputs(S, T, d, nb, dtype)
    o, lse, _ = pipeline.hash_forward(q, k, v, bucket, bucket, nb, 0.125, need_bwd=False)
    few = torch.tensor([0, 1, S // 2, S - 2, S - 1], device="cuda")
    o1, lse1, _ = pipeline.hash_forward(q[few], k[few], v[few], bucket[few], bucket[few], nb, 0.125, need_bwd=False)
    assert torch.equal(o[few], o1) and torch.equal(lse[few], lse1)
    # the first row sees itself alone (bf16: through fp16, whose smallest numbers are 2^-24 apart)
    assert torch.allclose(o[:, :, 0].float(), v[:, :, 0].float(), rtol=0, atol=0 if dtype == torch.float32 else 2.0 ** -24)


def test_backward_beyond_one_grid():
    S, T, d, nb = 33000, 2, 64, 256              # 33000 x (257 + 257) items of 256 threads
    (q, k, v, do), bucket = _inputs(S, T, d, nb, torch.bfloat16)
    _, _, ctx = pipeline.hash_forward(q, k, v, bucket, bucket, nb, 0.125)
    got = pipeline.hash_backward(ctx, do)
    few = torch.tensor([0, 1, S // 2, S - 2, S - 1], device="cuda")
    _, _, ctx1 = pipeline.hash_forward(q[few], k[few], v[few], bucket[few], bucket[few], nb, 0.125)
    want = pipeline.hash_backward(ctx1, do[few])
    for name, a, b in zip(("dQ", "dK", "dV"), got, want):
        assert torch.equal(a[few], b), name
