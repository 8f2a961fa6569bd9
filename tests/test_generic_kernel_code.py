"""The machine code of the shape-agnostic kernels: the loads of a step are under way together, and nothing is kept in scratch memory."""
import pytest

from test_kernel_waits import _named, built  # noqa: F401


def most_loads_under_way(code):
    """The longest run of loads that no branch and no wait for a load interrupts."""
    best = run = 0
    for _, op, args, target in code:
        if op.startswith("global_load"):
            run += 1
            best = max(best, run)
        elif target is not None or (op == "s_waitcnt" and "vmcnt" in args):
            run = 0
    return best


# at least: a GEMM operand's four elements of a row; attention: a piece of K and the elements of V across its rows; ... of q and d_o, and the statistics
@pytest.mark.parametrize("part,instances,loads", [("14gemm_generic_k", 18, 4), ("18attn_fwd_generic_k", 24, 5), ("17attn_dq_generic_k", 20, 5),
                                                  ("18attn_dkv_generic_k", 14, 17)])
def test_loads_of_a_step_are_under_way_together(built, part, instances, loads):  # noqa: F811
    """One wait per element or per pair of 16-wide pieces made a step of the GEMM up to 2.5 times, 64 keys of a 256-wide head 3 times as long."""
    found = _named(built, (part,))
    assert len(found) == instances
    few = {n: most_loads_under_way(c) for n, c in found.items() if most_loads_under_way(c) < loads}
    assert not few, few


def test_nothing_is_kept_in_scratch(built):  # noqa: F811
    """dQ of heads of more than 128 elements kept 74 registers there."""
    found = _named(built, ("_generic_k",))
    bad = [n for n, c in found.items() if any(op.startswith("scratch_") for _, op, _, _ in c)]
    assert len(found) == 76 and not bad, bad
