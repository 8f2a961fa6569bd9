"""The LM head's products over spans of several chunks (numerator form: all of them; fp32 logits: dh) against the fp64 oracle: spans of two to eight
chunks, last chunks and spans of a few rows or none that is active, and buffers that do not hold a span (back to one chunk at a time)."""
import numpy as np
import pytest
import torch

from oracle import head as o_head
from paper_2506_03077_amd import binding as sb
from paper_2506_03077_amd import synth

from gpu_util import TOL, assert_close, dev, host
from test_gpu_parity_small import head_case

pytestmark = pytest.mark.gpu

BF16 = dict(dtype="bf16", hidden=64, n_q_heads=4, n_kv_heads=2, head_dim=64, mlp_width=512)
F32 = dict(BF16, dtype="f32")


@pytest.mark.parametrize("objective,grad", [("sft", "f32"), ("grpo", "bf16"), ("dpo", "f32")])
@pytest.mark.parametrize("cfg", [dict(BF16, vocab=4096), dict(BF16, vocab=4093), dict(BF16, vocab=72), dict(BF16, hidden=1024, vocab=1096)])
@pytest.mark.parametrize("T,chunk,rows", [(260, 64, 0), (300, 70, 140), (129, 64, 128)])
def test_bf16_spans(cfg, T, chunk, rows, objective, grad):
    head_case(cfg, 2, T, chunk, objective, grad_dtype=grad, dw_group_rows=rows)


@pytest.mark.parametrize("vocab", [512, 37])
@pytest.mark.parametrize("T,chunk,rows", [(260, 64, 0), (300, 70, 140), (1000, 7, 0)])
def test_f32_spans(vocab, T, chunk, rows):
    head_case(dict(F32, vocab=vocab), 1, T, chunk, "sft", dw_group_rows=rows)


@pytest.mark.parametrize("vocab", [4096, 4093])
@pytest.mark.parametrize("active", [0, 1, 64, 129])
def test_chunks_and_spans_without_active_rows(vocab, active):
    T, cfg = 300, dict(BF16, vocab=vocab)
    inp = synth.head_inputs(cfg, seed=3, seq_len=T, vocab=vocab)
    tg = np.array(inp["targets"])
    tg[...] = np.abs(tg)                       # (all active ...)
    tg.reshape(-1)[active:] = -1               # ... but for the last rows
    ref = o_head.sft(inp["h"], inp["w"], tg, 1.0 / 64)
    hc = sb.head_cfg(sb.SBP_BF16, 1, T, 64, cfg["hidden"], vocab, sb.SBP_OBJ_SFT, 1.0 / 64, dw_group_rows=128)
    dh, dw, loss, n_active = sb.streambp_lmhead_ce_backward(hc, dev(inp["w"], "bf16"), dev(inp["h"], "bf16"), torch.from_numpy(tg).cuda())
    torch.cuda.synchronize()
    assert int(n_active.item()) == active == ref["n_active"]
    assert bool((dh.reshape(T, -1)[active:] == 0).all())
    if active == 0:
        assert bool((dw == 0).all()) and float(loss.item()) == 0.0
        return
    assert_close(host(dh), ref["dh"], TOL["bf16"], "dh")
    assert_close(host(dw), ref["dw"], TOL["bf16"], "dw")
    assert abs(float(loss.item()) - ref["loss"]) <= 1e-4 * abs(ref["loss"])
