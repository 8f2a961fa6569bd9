"""The shape-agnostic GEMM on rows that start anywhere (views with odd strides and offsets), in both storage types, at the edges of its steps, against fp64."""
import pytest
import torch

from paper_2506_03077_amd import binding as sb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("ta,tb", [(False, True), (False, False), (True, False)])
@pytest.mark.parametrize("M,N,K,pad,off", [(1, 1, 16, 1, 1), (33, 31, 17, 0, 0), (40, 33, 128, 3, 1), (70, 37, 127, 2, 2), (32, 65, 145, 5, 3), (31, 32, 515, 1, 1)])
def test_rows_that_start_anywhere(M, N, K, pad, off, ta, tb, dtype):
    gen = torch.Generator(device="cuda").manual_seed(M + N + K + pad)

    def view(rows, cols):
        return torch.randn((rows, cols + pad + off), generator=gen, device="cuda").to(dtype)[:, off:off + cols]

    A, B = view(*((K, M) if ta else (M, K))), view(*((N, K) if tb else (K, N)))
    C = torch.full((M, N), float("nan"), device="cuda")
    sb.debug_force_generic(gemm=True)
    try:
        code = sb.SBP_BF16 if dtype == torch.bfloat16 else sb.SBP_F32
        assert sb.lib().streambp_debug_gemm(M, N, K, int(ta), int(tb), code, sb.SBP_F32, 0, A.data_ptr(), B.data_ptr(), C.data_ptr(), A.stride(0), B.stride(0),
                                            N, None, 0, torch.cuda.current_stream().cuda_stream, None, None, None) == 0
    finally:
        sb.debug_force_generic()
    a, b = A.double(), B.double()
    want = (a.t() if ta else a) @ (b.t() if tb else b)
    bound = (K + 1) * 2.0 ** -23 * max(1.0, K ** 0.5) + 1e-6        # K ulp of the typical sum of K products
    assert bool(((C.double() - want).abs() <= bound).all())
