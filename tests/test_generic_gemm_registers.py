"""Registers of the shape-agnostic GEMM in the machine code that was built: three workgroups of eight waves share a CU, six waves a SIMD of 512 registers in
steps of eight.  With 82 of them two did, and an fp32 product of 2816 tiles of one step each took 19.5 us instead of 15.0."""
import re

from test_kernel_waits import _named, built  # noqa: F401


def registers(code, letter):
    """One more than the highest register of that letter that an instruction names."""
    most = 0
    for _, _, args, _ in code:
        for first, last in re.findall(rf"(?<![\w.]){letter}(?:(\d+)|\[\d+:(\d+)\])", args):
            most = max(most, 1 + int(first or last))
    return most


def test_three_workgroups_share_a_cu(built):  # noqa: F811
    found = _named(built, ("14gemm_generic_k",))
    assert len(found) == 18
    # (accumulation registers follow the vector registers, from a multiple of four on)
    used = {n: -(-registers(c, "v") // 4) * 4 + registers(c, "a") for n, c in found.items()}
    assert max(used.values()) <= 512 // 6 // 8 * 8, used
