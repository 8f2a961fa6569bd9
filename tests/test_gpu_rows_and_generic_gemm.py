"""The RMSNorm kernels at the edges of their row widths, the shape-agnostic GEMM at the edges of its tiles and reduction steps, and
weight-gradient groups that span short sequences - against fp64."""
import pytest
import torch

from paper_2506_03077_amd import binding as sb

from test_gpu_parity_small import MID16, run_layer_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("rows,d", [(1, 8), (5, 504), (3, 512), (4, 520), (6, 1024), (7, 1536), (9, 2056), (3, 2560), (4, 3072),
                                    (2, 3584), (6, 3592), (5, 4096), (3, 4104), (9, 5000)])
def test_rmsnorm_row_widths(rows, d, dtype):
    gen = torch.Generator(device="cuda").manual_seed(d + rows)
    x, dy = (torch.randn((rows, d), generator=gen, device="cuda").to(dtype) for _ in range(2))
    g = (1 + 0.1 * torch.randn(d, generator=gen, device="cuda")).to(dtype)
    y = sb.streambp_rmsnorm_forward(x, g, 1e-6)
    dx, dg = sb.streambp_rmsnorm_backward(x, g, dy, 1e-6)
    X, G, DY = x.double(), g.double(), dy.double()
    r = (X.square().mean(1, keepdim=True) + 1e-6).rsqrt()
    u = DY * G
    want = (X * r * G, u * r - X * r ** 3 * (u * X).mean(1, keepdim=True), (DY * X * r).sum(0))
    # fp32 arithmetic with sums of up to 4104 terms: 1e-5 of the largest value; bf16 results rounded once more (2^-8 with a tie)
    for got, ref, rounded in zip((y, dx, dg), want, (True, True, False)):
        bound = 1e-5 * float(ref.abs().max()) + (ref.abs() * 2.0 ** -8 if rounded and dtype == torch.bfloat16 else 0.0)
        assert bool(((got.double() - ref).abs() <= bound).all())


@pytest.mark.parametrize("ta,tb", [(False, True), (False, False), (True, False)])
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (31, 33, 15), (32, 32, 16), (33, 31, 17), (5, 70, 127), (64, 65, 130), (100, 36, 516)])
@pytest.mark.parametrize("acc", [False, True])
def test_generic_gemm_fp32(M, N, K, ta, tb, acc):
    gen = torch.Generator(device="cuda").manual_seed(M * 100 + N + K)
    A = torch.randn((K, M) if ta else (M, K), generator=gen, device="cuda")
    B = torch.randn((N, K) if tb else (K, N), generator=gen, device="cuda")
    C = torch.full((M, N), 0.5 if acc else float("nan"), device="cuda")
    assert sb.debug_gemm(A, B, C, M, N, K, ta, tb, acc=acc) == 0
    a, b = A.double(), B.double()
    want = (a.t() if ta else a) @ (b.t() if tb else b) + (0.5 if acc else 0.0)
    bound = (K + 1) * 2.0 ** -23 * max(1.0, K ** 0.5) + 1e-6        # K ulp of the typical sum of K products
    assert bool(((C.double() - want).abs() <= bound).all())


@pytest.mark.parametrize("T,chunk,batch", [(70, 64, 5), (130, 200, 9)])
def test_weight_gradient_groups_span_short_sequences(T, chunk, batch):
    run_layer_case(MID16, T, chunk, batch=batch, seed=6)                                                # default: up to three sequences a pass, two passes a launch
    run_layer_case(dict(MID16, mlp_width=128), T, chunk, batch=batch, seed=6, dw_group_rows=4 * chunk)     # MLP narrower than hidden: up to two
