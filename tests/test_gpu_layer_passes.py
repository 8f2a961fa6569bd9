"""How a layer call deals its rows to passes: several sequences at once with a last pass of fewer, a sequence in uneven parts, groups of passes that
share a weight-gradient launch - backward and forward against the fp64 oracle, with and without front padding and a window.  That the calls are
dealt so test_layer_plans.py reads off the host layer."""
import numpy as np
import pytest
import torch

from oracle import layer as o_layer
from paper_2506_03077_amd import binding as sb
from paper_2506_03077_amd import synth

from gpu_util import TOL, assert_close, dev, host, lib_layer_cfg, oracle_cfg
from layer_plan_cases import GROUPS, PASSES
from test_gpu_parity_small import run_layer_case

pytestmark = pytest.mark.gpu

@pytest.mark.parametrize("cfg,B,T,chunk,group,window,first", [c[:7] for c in PASSES])
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


@pytest.mark.parametrize("cfg,B,T,chunk,group", [c[:5] for c in GROUPS])
def test_passes_that_share_a_launch_of_bf16_weight_gradients_vs_oracle(cfg, B, T, chunk, group):
    run_layer_case(cfg, T, chunk, batch=B, grad_dtype="bf16", dw_group_rows=group)
