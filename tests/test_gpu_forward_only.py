"""Forward passes without a backward: the kernel fetches its own queries and no permuted copy of them is kept."""
import pytest
import torch

from paper_2306_01160_amd import binding as sc
from paper_2306_01160_amd import pipeline

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("variant,B,H,T,nb", [("hash", 1, 2, 300, 4), ("hash", 1, 2, 4096, 2), ("hash", 1, 3, 5003, 32),
                                               ("hash", 4, 12, 4097, 16), ("qkdrop", 1, 2, 2048, 1), ("qkdrop", 3, 4, 6001, 1)])
def test_outputs_equal_those_of_a_pass_with_backward(variant, B, H, T, nb, d):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(T + d)
    q, k, v = (torch.randn((B, H, T, d), device="cuda", generator=gen).to(torch.bfloat16) for _ in range(3))
    if variant == "hash":
        lq, lk = (torch.randint(0, nb, (B, H, T), device="cuda", generator=gen, dtype=torch.int32) for _ in range(2))
        run = lambda need: pipeline.hash_forward(q, k, v, lq, lk, nb, 0.125, need_bwd=need)  # noqa: E731
    else:
        lq, lk = ((torch.rand((B, H, T), device="cuda", generator=gen) < 0.5).to(torch.uint8) for _ in range(2))
        run = lambda need: pipeline.qkdrop_forward(q, k, v, lq, lk, 0.125, need_bwd=need)  # noqa: E731
    (o, lse, ctx), (o1, lse1, ctx1) = run(False), run(True)
    assert torch.equal(o, o1) and torch.equal(lse, lse1)
    n_k = None if variant == "hash" else ctx.n_k.tolist()
    assert ctx.q_p is None and ctx.bwd_work is None and ctx.o_f16 is None
    for name in ("k_p", "v_p"):
        a, b = getattr(ctx, name), getattr(ctx1, name)
        for s in range(B * H):
            n = T if n_k is None else n_k[s]
            assert torch.equal(a[s, :n], b[s, :n]), name


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("variant,nb", [(sc.SCFA_HASH, 8), (sc.SCFA_QKDROP, 1)])
def test_workspace_holds_no_query_rows(variant, nb, d):
    S, T = 6, 1000
    total, at = sc.scfa_forward_workspace(variant, S, T, d, nb, sc.SCFA_BF16, False)
    assert "q_perm" not in at and "k_perm" in at and "v_perm" in at
    with_bwd, at = sc.scfa_forward_workspace(variant, S, T, d, nb, sc.SCFA_BF16, True)
    assert "q_perm" in at and with_bwd - total >= 2 * 2 * S * T * d       # query rows and the fp16 copy of O
    assert "q_perm" in sc.scfa_forward_workspace(variant, S, T, d, nb, sc.SCFA_F16, False)[1]
