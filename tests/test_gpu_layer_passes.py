"""How a layer call deals its rows to passes: several sequences at once with a last pass of fewer, a sequence in uneven parts, groups of passes that
share a weight-gradient launch - backward and forward against the fp64 oracle, with and without front padding and a window."""
import numpy as np
import pytest
import torch

from oracle import layer as o_layer
from paper_2506_03077_amd import binding as sb
from paper_2506_03077_amd import synth

from gpu_util import TOL, assert_close, dev, host, lib_layer_cfg, oracle_cfg

pytestmark = pytest.mark.gpu

MID16 = dict(dtype="bf16", hidden=256, n_q_heads=4, n_kv_heads=2, head_dim=128, mlp_width=512)
NARROW = dict(dtype="bf16", hidden=256, n_q_heads=4, n_kv_heads=2, head_dim=64, mlp_width=64)      # an MLP that has no room for the rows of the K/V pass
TINY = synth.CONFIGS["tiny"]


@pytest.mark.parametrize("cfg,B,T,chunk,group,window,first", [
    (MID16, 5, 130, 64, 0, 0, [0, 129, 7, 130, 64]),    # two sequences, two, one
    (MID16, 7, 100, 100, 250, 0, None),                 # one sequence a pass, two passes a weight-gradient launch, forward two a pass
    (MID16, 2, 333, 64, 1, 50, [0, 70]),                # four parts of a sequence
    (NARROW, 3, 257, 64, 1, 0, None),
    (TINY, 5, 50, 40, 0, 16, [3, 0, 50, 49, 1]),        # three sequences, two
    (TINY, 2, 200, 40, 1, 0, None),
])
def test_passes_of_a_layer_vs_oracle(cfg, B, T, chunk, group, window, first):
    cfg, dt = dict(cfg, window=window), cfg["dtype"]
    inp = synth.layer_inputs(cfg, seed=11, seq_len=T, batch=B)
    _, dx_ref, g_ref = o_layer.layer_forward_backward(inp["x"], inp["w"], oracle_cfg(cfg), inp["dy"], first)
    w, x = {k: dev(v, dt) for k, v in inp["w"].items()}, dev(inp["x"], dt)
    lc = lib_layer_cfg(cfg, T, chunk, B, dw_group_rows=group, seq_first=first)
    dx, dw = sb.streambp_layer_backward(lc, w, x, dev(inp["dy"], dt))
    y = sb.streambp_layer_forward(lc, w, x)
    torch.cuda.synchronize()
    assert_close(host(dx), dx_ref, TOL[dt], "dx")
    for n in sb.WEIGHT_NAMES:
        assert_close(host(dw[n]), g_ref[n], TOL[dt], f"d{n}")
    y_ref = np.stack([o_layer.layer_forward(inp["x"][b], inp["w"], dict(oracle_cfg(cfg), first_valid=first[b] if first else 0))[0] for b in range(B)])
    assert_close(host(y), y_ref, TOL[dt], "y")
