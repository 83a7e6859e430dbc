"""Every item of every segment is done once, whatever the number of segments is to the 8 XCDs: fewer than 8, a multiple, one less
and one more, and odd ones whose ranks are turned; one launch for both gradients, and one each (which the event timers ask for), whose
bits are the same; tolerances as in test_gpu_attention_parity.py."""
import pytest
import torch

from gpu_util import assert_within, compare_backward, compare_forward, run_gpu
from paper_2306_01160_amd import binding as sc
from paper_2306_01160_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S", [1, 3, 7, 8, 9, 13, 15, 16, 17, 23])
@pytest.mark.parametrize("T,d,nb", [(300, 64, 5), (300, 128, 1)])
def test_segments_and_xcds(S, T, d, nb):
    wl = W.hash_uniform(7300 + S, 1, S, T, d, nb)
    o, lse, grads, _ = run_gpu(wl)
    assert_within(compare_forward(wl, o, lse), wl.dtype)
    assert_within(compare_backward(wl, grads), wl.dtype)
    sc.scfa_prof_reset()
    sc.scfa_prof_enable(True)
    try:
        apart = run_gpu(wl)[2]
        assert sc.scfa_prof_read("bwd_dkdv")[1] == 1 and sc.scfa_prof_read("bwd_dq")[1] == 1
    finally:
        sc.scfa_prof_enable(False)
        sc.scfa_prof_reset()
    for name, a, b in zip(("dQ", "dK", "dV"), grads, apart):
        assert torch.equal(a, b), name
