"""The LM head whose weight gradient reads h transposed (outputs of 10^8 elements and more) against the fp64 oracle, and the GEMM form that it uses."""
import pytest

from test_gpu_gemm_edges import _check, _operands
from test_gpu_parity_small import head_case

pytestmark = pytest.mark.gpu

CFG = dict(dtype="bf16", n_q_heads=4, n_kv_heads=2, head_dim=64, mlp_width=512)


@pytest.mark.parametrize("grad", ["f32", "bf16"])
@pytest.mark.parametrize("K", [64, 128, 192, 320])
@pytest.mark.parametrize("M,N", [(8, 1), (120, 127), (264, 257), (520, 400)])
def test_both_operands_transposed(K, M, N, grad):
    import torch
    from paper_2506_03077_amd import binding as sb
    N = -(-N // 8) * 8
    A, B, want = _operands(M, N, K, True, True)
    C = torch.zeros(M, N, dtype=torch.bfloat16 if grad == "bf16" else torch.float32, device="cuda")
    assert sb.debug_gemm(A, B, C, M, N, K, True, True, acc=True) == 1
    _check(C, want, K)


@pytest.mark.parametrize("hidden,vocab", [(16384, 6107), (16384, 6112), (4096, 24424)])      # fp32 logits; numerators chunk by chunk; numerators in spans
@pytest.mark.parametrize("T,chunk,group", [(1, 64, 0), (65, 64, 0), (200, 65, 0), (200, 65, 130), (130, 63, 63)])
def test_head_with_transposed_rows(T, chunk, group, hidden, vocab):
    # a chunk of one row, chunks one row longer and shorter than the transposed copy's 64-column tiles, groups of every size; some rows are ignored
    head_case(dict(CFG, hidden=hidden, vocab=vocab), 1, T, chunk, "sft", loss_scale=1.0 / max(1, T), dw_group_rows=group, grad_dtype="f32" if T != 130 else "bf16")
