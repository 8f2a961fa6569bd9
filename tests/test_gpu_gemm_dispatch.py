"""Which kernels a layer of few output tiles runs on, by launches counted around the oracle comparison, and the accumulate form with both operands
reduction-major on an output that holds something already."""
import pytest
import torch

from paper_2506_03077_amd import binding as sb

from test_gpu_gemm_edges import _check, _operands
from test_gpu_parity_small import MID16, run_layer_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grad", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("M,N,K", [(8, 8, 64), (264, 272, 192), (520, 400, 320)])
def test_both_operands_transposed_add_to_what_is_there(M, N, K, grad):
    A, B, want = _operands(M, N, K, True, True)
    start = torch.randn((M, N), generator=torch.Generator(device="cuda").manual_seed(5), device="cuda").to(grad)
    C = start.clone()
    assert sb.debug_gemm(A, B, C, M, N, K, True, True, acc=True) == 1
    _check(C, want + start.double().cpu(), K)


# one pass: q, K and V in one launch, o, gate with up, dact, dm (two operand pairs), do, da (three segments)
@pytest.mark.parametrize("cfg,T,few", [(MID16, 640, 7), (dict(MID16, hidden=1024, head_dim=128, mlp_width=1408), 300, 7)])
def test_a_layer_of_few_tiles_runs_on_their_kernels(cfg, T, few):
    sb.debug_profile_begin()
    try:
        run_layer_case(cfg, T, T)
    finally:
        counts = {k: v["count"] for k, v in sb.debug_profile_end().items() if v["count"]}
    assert counts.get("gemm_few_k", 0) == few, counts
