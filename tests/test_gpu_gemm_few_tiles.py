"""C += of the weight-gradient form on both sides of 32 output tiles, up to which C goes through the caches: whole and ragged tiles, few and many K steps, rows of C
further apart than they are long, with and without room for partial tiles, twice in a row, against fp64."""
import pytest

from test_gpu_gemm_edges import _check, _operands

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N", [(8, 8), (264, 136), (2048, 1024), (2040, 1016), (2304, 1024), (2056, 1032)])      # 1, 2, 32, 32, 36, 45 tiles
@pytest.mark.parametrize("K", [64, 333, 2120])
@pytest.mark.parametrize("room", [False, True])
def test_accumulate(room, K, M, N):
    import torch
    from paper_2506_03077_amd import binding as sb
    A, B, want = _operands(M, N, K, True, False)
    wide = torch.full((M, N + 8), float("nan"), device="cuda")
    C = wide[:, :N]
    C.fill_(1.0)
    scratch = torch.empty(64 << 20, dtype=torch.uint8, device="cuda") if room else None
    for times in (1, 2):
        assert sb.debug_gemm(A, B, C, M, N, K, True, False, acc=True, scratch=scratch) == 1
        _check(C, 1.0 + times * want, 2 * K)
    assert bool(torch.isnan(wide[:, N:]).all())
