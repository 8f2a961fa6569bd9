"""The machine code of dQ and dK/dV in one launch, heads of up to 64 elements: a query block's four statistics and its elements of d_o and q across four rows are
loaded together, nothing is kept in scratch."""
from test_generic_kernel_code import most_loads_under_way
from test_kernel_waits import _named, built  # noqa: F401


def test_one_launch_backward(built):  # noqa: F811
    found = _named(built, ("17attn_bwd_narrow_k",))
    assert len(found) == 8
    assert not [n for n, c in found.items() if any(op.startswith("scratch_") for _, op, _, _ in c) or most_loads_under_way(c) < 12]
