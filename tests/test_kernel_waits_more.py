"""The waits of further kernels whose LDS is refilled by direct-to-LDS loads, walked as in test_kernel_waits: the attention backward in one
launch and the GEMM for outputs of few tiles consume every fragment (or wait for it) within the slot in which it is read."""
import pytest

from test_kernel_waits import _named, barriers_passed_unwaited, built  # noqa: F401


@pytest.mark.parametrize("part,instances", [("15attn_bwd_mfma_k", 4), ("10gemm_few_k", 12)])
def test_reads_are_waited_for_within_the_slot(built, part, instances):  # noqa: F811
    found = _named(built, (part,))
    assert len(found) == instances
    worst = {n: barriers_passed_unwaited(c) for n, c in found.items()}
    assert max(worst.values()) == 0, {n: w for n, w in worst.items() if w}


def test_shares_taken_without_a_break_have_kernels_that_keep_the_schedule(built):  # noqa: F811
    """dK/dV without room for the sums of its shares: a loop around the pipeline refilled it for every share (143 -> 228 us for 512 queries)."""
    found = _named(built, ("18attn_bwd_in_turn_k",))
    assert len(found) == 4
    worst = {n: barriers_passed_unwaited(c) for n, c in found.items()}
    assert max(worst.values()) == 0, {n: w for n, w in worst.items() if w}


def test_shared_last_rounds_keep_the_gemm_schedule(built):  # noqa: F811
    found = _named(built, ("18gemm_mfma_shared_k",))
    assert len(found) == 2
    worst = {n: barriers_passed_unwaited(c) for n, c in found.items()}
    assert max(worst.values()) <= 2, {n: w for n, w in worst.items() if w > 2}
