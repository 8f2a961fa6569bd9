"""The MFMA GEMM's main loop at the edges of its schedule: one to six K steps (the pipeline's prologue, its counted tail and the odd
step after the unrolled pair), ragged reductions, and output sizes around the 256-wide tile and its 128-row halves."""
import pytest

pytestmark = pytest.mark.gpu


def _operands(M, N, K, ta, tb):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(M * 7919 + N * 31 + K)
    r = lambda *s: torch.randn(s, generator=g, device="cuda").bfloat16()
    A, B = (r(K, M) if ta else r(M, K)), (r(N, K) if tb else r(K, N))
    a, b = A.double().cpu(), B.double().cpu()
    return A, B, (a.t() if ta else a) @ (b.t() if tb else b)


def _check(C, want, K):
    """fp32 sums of K products of N(0, 1) values: error below K ulp of the typical sum sqrt(K) in any order (measured ~ sqrt(K)
    ulp); a bf16 result is rounded once more, 2^-8 relative to the value (2^-9 plus a flip at a tie)."""
    import torch
    got = C.double().cpu()
    bound = K * 2.0 ** -23 * max(1.0, K ** 0.5) + 1e-6
    if C.dtype == torch.bfloat16:
        bound = bound + want.abs() * 2.0 ** -8
    assert bool(torch.isfinite(got).all())
    assert bool(((got - want).abs() <= bound).all()), float((got - want).abs().max())


@pytest.mark.parametrize("layout", ["nt", "nn"])
@pytest.mark.parametrize("K", [64, 128, 192, 256, 320, 384])
@pytest.mark.parametrize("M,N", [(1, 8), (127, 120), (129, 136), (256, 256), (257, 264), (400, 520)])
def test_few_k_steps(layout, K, M, N):
    import torch
    from paper_2506_03077_amd import binding as sb
    A, B, want = _operands(M, N, K, False, layout == "nt")
    for dt in (torch.float32, torch.bfloat16):
        C = torch.full((M, N), float("nan"), dtype=dt, device="cuda")
        assert sb.debug_gemm(A, B, C, M, N, K, False, layout == "nt") == 1
        _check(C, want, K)


@pytest.mark.parametrize("K", [1, 8, 31, 32, 33, 63, 64, 65, 96, 127, 128, 129, 160, 191, 192, 193, 255, 320, 333])
@pytest.mark.parametrize("M,N", [(8, 8), (128, 264), (264, 136)])
def test_ragged_reduction_of_the_weight_gradient_form(K, M, N):
    import torch
    from paper_2506_03077_amd import binding as sb
    A, B, want = _operands(M, N, K, True, False)
    # rows past the reduction's end hold NaN: none may be read
    A2 = torch.full((K + 64, M), float("nan"), dtype=torch.bfloat16, device="cuda"); A2[:K] = A
    B2 = torch.full((K + 64, N), float("nan"), dtype=torch.bfloat16, device="cuda"); B2[:K] = B
    C = torch.ones((M, N), dtype=torch.float32, device="cuda")
    assert sb.debug_gemm(A2, B2, C, M, N, K, True, False, acc=True) == 1
    _check(C, want + 1.0, K)
    Cb = torch.ones((M, N), dtype=torch.bfloat16, device="cuda")
    assert sb.debug_gemm(A2, B2, Cb, M, N, K, True, False, acc=True) == 1
    _check(Cb, want + 1.0, K)


@pytest.mark.parametrize("Ks", [(40, 64), (64, 200, 8), (129, 1, 63, 64)])
def test_segments_of_unequal_length(Ks):
    import torch
    from paper_2506_03077_amd import binding as sb
    M, N = 264, 136
    ops = [_operands(M, N, k, True, False) for k in Ks]
    C = torch.zeros((M, N), dtype=torch.float32, device="cuda")
    assert sb.debug_gemm_dw_segments([o[0] for o in ops], [o[1] for o in ops], C, M, N, list(Ks)) == 1
    _check(C, sum(o[2] for o in ops), sum(Ks))


@pytest.mark.parametrize("M,N,K", [(72, 72, 64), (256, 264, 128)])
@pytest.mark.parametrize("ta,tb,acc", [(False, True, False), (False, False, False), (True, False, True)])
def test_rows_of_c_that_start_between_16_byte_boundaries(M, N, K, ta, tb, acc):
    """C a column slice whose rows lie N + 4 elements apart: 16-byte aligned in fp32 (MFMA kernels), 8-byte aligned in bf16, where the
    MFMA kernels' 16-byte accesses do not fit."""
    import torch
    from paper_2506_03077_amd import binding as sb
    A, B, want = _operands(M, N, K, ta, tb)
    for dt, mfma in ((torch.float32, 1), (torch.bfloat16, 0)):
        wide = torch.full((M, N + 4), 3.0, dtype=dt, device="cuda")
        C = wide[:, :N]
        C.fill_(1.0)
        assert sb.debug_gemm(A, B, C, M, N, K, ta, tb, acc=acc) == mfma
        _check(C, want + (1.0 if acc else 0.0), K)
        assert bool((wide[:, N:] == 3.0).all())


# (M, N, K, layout, accumulate, tiles, splits): as many ways as the scratch of a whole chip lets the schedule take.  27 slices of 5
# K steps leave two of 128 steps (one slice ragged, one empty); 15 of 13 leave the last with 10; 27 of 125 ragged steps two empty ones.
@pytest.mark.parametrize("M,N,K,layout,acc,tiles,splits,out", [
    (256, 256, 8192, "nt", False, 1, 27, "f32"), (256, 256, 8192, "nt", False, 1, 27, "bf16"), (40, 256, 8192, "nn", False, 1, 27, "f32"),
    (40, 256, 8192, "nn", False, 1, 27, "bf16"), (40, 264, 8192, "nt", True, 2, 27, "f32"), (512, 1024, 12288, "nt", False, 8, 15, "f32"),
    (512, 1024, 12288, "nt", False, 8, 15, "bf16"), (264, 256, 7993, "tn", True, 2, 27, "f32")])
def test_reductions_split_more_than_eight_ways(M, N, K, layout, acc, tiles, splits, out):
    import torch
    from paper_2506_03077_amd import binding as sb
    A, B, want = _operands(M, N, K, layout == "tn", layout == "nt")
    scratch = torch.full((256 * 256 * 256,), float("nan"), device="cuda")
    C = torch.ones((M, N), dtype=torch.float32 if out == "f32" else torch.bfloat16, device="cuda")
    assert sb.debug_gemm(A, B, C, M, N, K, layout == "tn", layout == "nt", acc=acc, scratch=scratch) == 1
    _check(C, want + (1.0 if acc else 0.0), K)
    # one partial tile per tile and slice: 256 columns, of an output of fewer than 256 rows only those rows
    assert int(torch.isfinite(scratch).sum()) == splits * tiles * min(M, 256) * 256


def test_two_operand_pairs_with_slices_across_their_boundary():
    """C = A B + A2 B2 as one reduction of 34 K steps, split seven ways: slice 3 takes steps 15 .. 19, of which 17 on are the second pair's."""
    import torch
    from paper_2506_03077_amd import binding as sb
    M, N, K = 300, 512, 1088
    A, B, first = _operands(M, N, K, False, False)
    A2, B2, _ = _operands(M, N, K + 64, False, False)      # other values
    A2, B2 = A2[:, :K].contiguous(), B2[:K].contiguous()
    second = A2.double().cpu() @ B2.double().cpu()
    scratch = torch.full((256 * 256 * 256,), float("nan"), device="cuda")
    C = torch.full((M, N), float("nan"), device="cuda")
    assert sb.debug_gemm(A, B, C, M, N, K, False, False, scratch=scratch, A2=A2, B2=B2) == 1
    _check(C, first + second, 2 * K)
    assert int(torch.isfinite(scratch).sum()) == 7 * 4 * 256 * 256
