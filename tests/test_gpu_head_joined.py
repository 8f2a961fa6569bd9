"""The head's weight gradient as one reduction over all units of a group, whose last round of tiles is split by the number of active rows: from none to all,
in groups that end with a unit and inside one, fp32 and bf16 gradients, against the fp64 oracle."""
import numpy as np
import pytest
import torch

from oracle import head as o_head
from paper_2506_03077_amd import binding as sb
from paper_2506_03077_amd import synth

from gpu_util import TOL, assert_close, dev, host

pytestmark = pytest.mark.gpu

T, CHUNK, HIDDEN, VOCAB = 1100, 256, 1024, 16650      # 66 x 4 tiles: a round and eight more; a vocabulary that keeps fp32 logits, five units


@pytest.mark.parametrize("grad", ["f32", "bf16"])
@pytest.mark.parametrize("active,group", [(0, 0), (1, 0), (256, 0), (300, 512), (512, 512), (700, 512), (1100, 0), (1100, 768)])
def test_weight_gradient_of_a_group(active, group, grad):
    cfg = dict(dtype="bf16", hidden=HIDDEN, n_q_heads=4, n_kv_heads=2, head_dim=64, mlp_width=512)
    inp = synth.head_inputs(cfg, seed=8, seq_len=T, vocab=VOCAB)
    tg = np.abs(np.array(inp["targets"]))
    tg.reshape(-1)[active:] = -1
    ref = o_head.sft(inp["h"], inp["w"], tg, 1.0 / 64)
    hc = sb.head_cfg(sb.SBP_BF16, 1, T, CHUNK, HIDDEN, VOCAB, sb.SBP_OBJ_SFT, 1.0 / 64, dw_group_rows=group,
                     grad_dtype=sb.SBP_BF16 if grad == "bf16" else sb.SBP_F32)
    _, dw, _, n_active = sb.streambp_lmhead_ce_backward(hc, dev(inp["w"], "bf16"), dev(inp["h"], "bf16"), torch.from_numpy(tg).cuda())
    torch.cuda.synchronize()
    assert int(n_active.item()) == active
    if active == 0:
        assert bool((dw == 0).all())
    else:
        assert_close(host(dw), ref["dw"], TOL["bf16"], "dw")
