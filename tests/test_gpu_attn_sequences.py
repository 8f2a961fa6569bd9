"""Several sequences of a pass in one launch of the attention kernels: padding of their own, key blocks that some or all of them hide, windows, both
head sizes, the backward in one launch and in two, with and without sums of parts, a last pass of fewer sequences, against the fp64 oracle.  How many
sequences each pass takes, and which kernels its size picks, test_layer_plans.py reads off the host layer."""
import pytest
import torch

from oracle import layer as o_layer
from paper_2506_03077_amd import binding as sb
from paper_2506_03077_amd import synth

from gpu_util import TOL, assert_close, dev, host, lib_layer_cfg, oracle_cfg
from layer_plan_cases import SEQUENCES

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("c", SEQUENCES, ids=lambda c: f"{c['B']}x{c['T']}-{c['cfg']['n_q_heads']}-{c['cfg']['n_kv_heads']}-{c['cfg']['head_dim']}")
def test_sequences_share_the_attention_launches(c):
    cfg, B, T, first = c["cfg"], c["B"], c["T"], c["first"]
    inp = synth.layer_inputs(cfg, seed=5, seq_len=T, batch=B)
    _, dx_ref, g_ref = o_layer.layer_forward_backward(inp["x"], inp["w"], oracle_cfg(cfg), inp["dy"], first)
    w = {k: dev(v, "bf16") for k, v in inp["w"].items()}
    sb.debug_profile_begin()
    try:
        dx, dw = sb.streambp_layer_backward(lib_layer_cfg(cfg, T, T, B, seq_first=first), w, dev(inp["x"], "bf16"), dev(inp["dy"], "bf16"))
        torch.cuda.synchronize()
    finally:
        counts = {k: v["count"] for k, v in sb.debug_profile_end().items() if v["count"]}
    attn = {k: n for k, n in counts.items() if "attn" in k}
    assert len(attn) == 2 and set(attn.values()) == {len(c["passes"])}, counts
    assert_close(host(dx), dx_ref, TOL["bf16"], "dx")
    for n in sb.WEIGHT_NAMES:
        assert_close(host(dw[n]), g_ref[n], TOL["bf16"], f"d{n}")
