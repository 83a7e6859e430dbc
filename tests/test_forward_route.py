"""Which whole-pass forwards run in one launch: host arithmetic, no GPU.  The sizes are those that test_gpu_fp32_in_one.py runs, so that
its comparisons are of the two routes, and the ones on either side of the rule's limits."""
import pytest

from paper_2306_01160_amd import binding

HASH, DROP, F32 = binding.SCFA_HASH, binding.SCFA_QKDROP, binding.SCFA_F32


def _in_one(variant, S, T, d, nb, dtype=F32, need_bwd=False):
    return binding.scfa_prof_forward_in_one(variant, S, T, d, nb, dtype, need_bwd)


@pytest.mark.parametrize("S,T,d,nb", [
    (1, 1, 64, 1), (2, 1, 128, 3), (3, 63, 64, 2), (2, 64, 64, 1), (2, 65, 128, 4), (1, 256, 64, 256), (5, 129, 64, 3), (2, 1023, 64, 5),
    (1, 1024, 64, 7), (1, 1024, 128, 2), (85, 300, 64, 4), (85, 128, 128, 4), (2, 700, 64, 240), (1, 1000, 128, 240)])
def test_a_few_short_fp32_segments_take_one_launch(S, T, d, nb):
    assert _in_one(HASH, S, T, d, nb)
    assert not _in_one(HASH, S, T, d, nb, need_bwd=True)
    assert not _in_one(HASH, S, T, d, nb, dtype=binding.SCFA_BF16)


@pytest.mark.parametrize("S,T,d", [(1, 1, 64), (3, 200, 64), (3, 200, 128), (2, 1024, 64), (4, 777, 64)])
def test_a_few_short_segments_of_kept_tokens_take_one_launch(S, T, d):
    assert _in_one(DROP, S, T, d, 1)
    assert not _in_one(DROP, S, T, d, 1, need_bwd=True)


@pytest.mark.parametrize("variant,S,T,d,nb", [
    (HASH, 1, 1025, 64, 7), (DROP, 4, 1025, 64, 1),                               # longer than a workgroup sorts
    (HASH, 86, 300, 64, 4), (HASH, 86, 128, 128, 4), (HASH, 2, 1000, 128, 240)])  # more workgroups than are resident at once
def test_past_the_limits_they_do_not(variant, S, T, d, nb):
    assert not _in_one(variant, S, T, d, nb)


def test_the_timers_keep_the_launches_apart():
    binding.scfa_prof_enable(True)
    try:
        assert not _in_one(HASH, 1, 256, 64, 4)
    finally:
        binding.scfa_prof_enable(False)
    assert _in_one(HASH, 1, 256, 64, 4)


def test_sizes_that_the_forward_refuses():
    with pytest.raises(binding.ScfaError):
        _in_one(HASH, 1, 256, 96, 4)
    with pytest.raises(binding.ScfaError):
        _in_one(DROP, 1, 256, 64, 4)
