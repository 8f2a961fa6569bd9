"""The shape-agnostic attention kernels at the edges of their 16 x 16 blocks and of the head widths they have instances for, and with
infinities and NaN in rows that the mask hides; several problems and reduction segments per launch of the shape-agnostic GEMM."""
import numpy as np
import pytest
import torch

from oracle import attn as o_attn
from paper_2506_03077_amd import binding as sb

from gpu_util import TOL, assert_close, dev, host
from test_gpu_masks import masked_attn_case
from test_gpu_parity_small import run_layer_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("dh", [1, 2, 15, 16, 17, 32, 36, 62, 66, 128, 130, 256])
def test_head_widths(dtype, dh):
    if dtype == "bf16" and dh == 128:
        dh = 126                                   # (128 runs on the bf16 MFMA kernels)
    masked_attn_case(dtype, 4, 2, dh, 19, 21, 0, 0)


@pytest.mark.parametrize("hq,hkv,s,c,window,kv_first", [
    (1, 1, 0, 1, 0, 0), (2, 2, 0, 16, 0, 0), (2, 1, 0, 17, 0, 0), (4, 2, 15, 1, 0, 0), (4, 4, 16, 33, 16, 0), (3, 1, 100, 50, 1, 0),
    (6, 2, 0, 40, 0, 35), (4, 2, 300, 130, 37, 290), (2, 2, 1000, 5, 0, 0)])
def test_blocks_and_masks_f32(hq, hkv, s, c, window, kv_first):
    masked_attn_case("f32", hq, hkv, 16, s, c, window, kv_first)


@pytest.mark.parametrize("dtype,dh", [("f32", 16), ("f32", 80), ("bf16", 24)])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_hidden_rows_reach_nothing(dtype, dh, bad):
    """Keys 0 .. 4 are padding, the window hides keys from later queries, keys past a query are hidden by causality, and query row 0 sees no key:
    what they hold must not show where they are hidden."""
    hq, hkv, s, c, window, first = 4, 2, 11, 30, 9, 12
    rng = np.random.default_rng(3)
    r = lambda rows, heads: dev(rng.standard_normal((rows, heads, dh)), dtype)
    q, k, v, d_o = r(c, hq), r(s + c, hkv), r(s + c, hkv), r(c, hq)
    ac = sb.attn_cfg(sb.SBP_F32 if dtype == "f32" else sb.SBP_BF16, hq, hkv, dh, s, c, dh ** -0.5, window, first)
    o, lse = sb.streambp_attn_chunk_forward(ac, q, k, v)
    want = sb.streambp_attn_chunk_backward(ac, q, k, v, o, lse, d_o)
    k2, v2, q2, d2 = k.clone(), v.clone(), q.clone(), d_o.clone()
    k2[:first] = bad; v2[:first] = bad             # padding
    q2[0] = bad; d2[0] = bad                       # (position 11 sees no key)
    o2, lse2 = sb.streambp_attn_chunk_forward(ac, q2, k2, v2)
    assert torch.equal(lse, lse2) and torch.allclose(o.float(), o2.float(), rtol=1e-5, atol=1e-6)
    got = sb.streambp_attn_chunk_backward(ac, q2, k2, v2, o2, lse2, d2)
    for a, b in zip(want, got):
        assert_close(host(b), host(a), TOL[dtype], "hidden rows")
    # a key that only the last queries see: the others keep their bits
    v3 = v.clone(); v3[s + c - 1] = bad
    o3, lse3 = sb.streambp_attn_chunk_forward(ac, q, k, v3)
    assert torch.equal(lse, lse3) and torch.allclose(o[:-1].float(), o3[:-1].float(), rtol=1e-5, atol=1e-6)
    assert not bool(torch.isfinite(o3[-1].float()).all())


# two passes of a sequence and seven, widths that are no multiple of the GEMM's 32 x 32 tiles or 16-deep steps
@pytest.mark.parametrize("cfg,T,chunk,batch", [
    (dict(dtype="f32", hidden=40, n_q_heads=4, n_kv_heads=2, head_dim=10, mlp_width=53, vocab=64), 33, 20, 2),
    (dict(dtype="f32", hidden=65, n_q_heads=2, n_kv_heads=1, head_dim=34, mlp_width=129, vocab=64), 70, 8, 1),
    (dict(dtype="bf16", hidden=72, n_q_heads=6, n_kv_heads=2, head_dim=24, mlp_width=100, vocab=64), 90, 10, 1)])
def test_layer_on_the_shape_agnostic_kernels(cfg, T, chunk, batch):
    run_layer_case(cfg, T, chunk, batch=batch, seed=11, dw_group_rows=1)
