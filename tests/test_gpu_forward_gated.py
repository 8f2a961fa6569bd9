"""The chunked forward whose gate and up products leave as act = silu(gate) * up from one launch (from 200 output tiles on), against the fp64
oracle: ragged rows and a ragged last column tile, and the same rows through a chunk size that keeps the products apart."""
import pytest
import torch

from oracle import layer as o_layer
from paper_2506_03077_amd import binding as sb
from paper_2506_03077_amd import synth

from gpu_util import TOL, assert_close, dev, host, lib_layer_cfg, oracle_cfg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,chunk,mlp", [(300, 300, 12872), (600, 512, 12864)])
def test_layer_forward_with_many_gate_tiles(T, chunk, mlp):
    cfg = dict(dtype="bf16", hidden=128, n_q_heads=2, n_kv_heads=1, head_dim=64, mlp_width=mlp, vocab=64)
    inp = synth.layer_inputs(cfg, seed=5, seq_len=T)
    want = o_layer.layer_forward_backward(inp["x"], inp["w"], oracle_cfg(cfg), inp["dy"])[0]
    w = {k: dev(v, "bf16") for k, v in inp["w"].items()}
    x = dev(inp["x"], "bf16")
    got = sb.streambp_layer_forward(lib_layer_cfg(cfg, T, chunk), w, x)
    torch.cuda.synchronize()
    assert_close(host(got).reshape(want.shape), want, TOL["bf16"], "y")
    apart = sb.streambp_layer_forward(lib_layer_cfg(cfg, T, 64, dw_group_rows=1), w, x)      # (passes of 75 and 86 rows)
    assert_close(host(apart), host(got), TOL["bf16"], "chunk 64")
