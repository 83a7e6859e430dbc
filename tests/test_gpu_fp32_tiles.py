"""fp32 forward at the edges of its tiles: query tiles of 64 rows (two wavefronts of 32), key tiles of 32 walked by
two key splits that are put together at the end.

Tolerance: fp32 rounding of sums of at most 257 terms of O(1), as for the fp32 path elsewhere (1e-4 on O, 1e-5 on LSE)."""
import pytest

from paper_2306_01160_amd import workloads as W

from gpu_util import assert_within, compare_forward, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("strict", [False, True])
@pytest.mark.parametrize("T", [2, 31, 33, 64, 65, 127, 129, 257])
def test_fp32_forward_tile_edges(T, strict, d):
    for wl in (W.hash_uniform(T, 1, 3, T, d, 1, dtype="f32", passes="fwd"),
               W.hash_uniform(T + 1, 1, 3, T, d, 5, dtype="f32", passes="fwd"),
               W.qkdrop_bernoulli(T + 2, 1, 3, T, d, 0.7, 0.6, dtype="f32", passes="fwd")):
        wl.meta["strict"] = strict
        o, lse, _, _ = run_gpu(wl, backward=False)
        assert_within(compare_forward(wl, o, lse), "f32")
