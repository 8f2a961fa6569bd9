"""Several sequences of a pass in one launch of the attention kernels: padding of their own, key blocks that some or all of them hide, windows, both
head sizes, few and many workgroups, as many sequences as a launch takes and more, against the fp64 oracle."""
import pytest
import torch

from oracle import layer as o_layer
from paper_2506_03077_amd import binding as sb
from paper_2506_03077_amd import synth

from gpu_util import TOL, assert_close, dev, host, lib_layer_cfg, oracle_cfg

pytestmark = pytest.mark.gpu


def _cfg(hq, hkv, dh, window=0):
    return dict(dtype="bf16", hidden=256, n_q_heads=hq, n_kv_heads=hkv, head_dim=dh, mlp_width=512, window=window)


@pytest.mark.parametrize("cfg,B,T,first", [
    (_cfg(4, 2, 128), 3, 300, [130, 200, 299]),          # the first key block hidden by all, the second by one
    (_cfg(4, 2, 64), 4, 257, [0, 150, 256, 257]),        # a sequence without a visible key
    (_cfg(8, 2, 128, 100), 4, 400, None),
    (_cfg(4, 4, 64, 33), 5, 130, [0, 1, 2, 64, 129]),
    (_cfg(4, 2, 128), 33, 20, list(range(20)) + [0] * 13),
    (_cfg(32, 8, 64), 32, 128, None),                    # 1024 query tiles: dQ and dK/dV in launches of their own
])
def test_sequences_share_the_attention_launches(cfg, B, T, first):
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
    assert len(attn) == 2 and max(attn.values()) < B, counts
    assert_close(host(dx), dx_ref, TOL["bf16"], "dx")
    for n in sb.WEIGHT_NAMES:
        assert_close(host(dw[n]), g_ref[n], TOL["bf16"], f"d{n}")
