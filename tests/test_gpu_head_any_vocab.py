"""GPU parity of the bf16 LM head against the fp64 oracle at vocabularies of any size."""
import numpy as np
import pytest
import torch

from oracle import head as o_head
from paper_2506_03077_amd import binding as sb
from paper_2506_03077_amd import synth

from gpu_util import TOL, assert_close, dev, host
from test_gpu_parity_small import head_case

pytestmark = pytest.mark.gpu

CFG = dict(dtype="bf16", hidden=256, n_q_heads=4, n_kv_heads=2, head_dim=64, mlp_width=512, vocab=1024)


@pytest.mark.parametrize("vocab", [1, 7, 64, 255, 257, 333, 1021, 4099])
def test_head_bf16_any_vocabulary(vocab):
    before = sb.streambp_generic_launches()
    head_case(dict(CFG, vocab=vocab), 2, 300, 128, "sft", loss_scale=1.0 / 450)
    assert sb.streambp_generic_launches() == before


@pytest.mark.parametrize("objective,grad", [("grpo", "bf16"), ("dpo", "f32"), ("dpo", "bf16")])
def test_head_bf16_odd_vocabulary_objectives(objective, grad):
    head_case(dict(CFG, vocab=777), 2, 333, 100, objective, grad_dtype=grad)


@pytest.mark.parametrize("vocab", [776, 777, 1024])
def test_head_rows_of_very_different_scale(vocab):
    # every seventh row scaled so that its logits reach several hundred, every seventh shifted by -256: block maxima, padding columns
    # and neighbours in the same tile must not mix
    T = 400
    inp = synth.head_inputs(dict(CFG, vocab=vocab), seed=11, seq_len=T, vocab=vocab)
    h, w = np.array(inp["h"]), np.array(inp["w"])
    h[:, ::7] *= 512.0                       # (powers of two: still exact in bf16)
    w[:, 0] = 0.0625                         # one direction that all words share ...
    h[:, 3::7, 0] = -4096.0                  # ... along which all logits of these rows fall by 256
    # (Column 0 of dh is exactly zero - the rows of dz sum to zero - and rounding dz to bf16 moves it by up to coef * 2^-9 * 0.0625 *
    # sum(p) = 4e-7, a twentieth of the allowance of 2e-2 * max|dh| = 6.8e-6; shared weights of 1.0 would use all of it.)
    ref = o_head.sft(h, w, inp["targets"], 1.0 / 300)
    hc = sb.head_cfg(sb.SBP_BF16, 1, T, 128, 256, vocab, sb.SBP_OBJ_SFT, 1.0 / 300)
    dh, dw, loss, n_active = sb.streambp_lmhead_ce_backward(hc, dev(w, "bf16"), dev(h, "bf16"), torch.from_numpy(inp["targets"]).cuda())
    torch.cuda.synchronize()
    assert int(n_active.item()) == ref["n_active"]
    assert_close(host(dh), ref["dh"], TOL["bf16"], "dh")
    assert_close(host(dw), ref["dw"], TOL["bf16"], "dw")
    assert abs(float(loss.item()) - ref["loss"]) <= 1e-4 * abs(ref["loss"])
