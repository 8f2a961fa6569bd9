"""GPU parity of the MFMA attention kernels against the fp64 oracle: 64-wide heads (masked, ragged), whole 256-query tiles and the form
that splits the keys over the wave groups, a layer with 64-wide heads."""
import pytest
import torch

from paper_2506_03077_amd import binding as sb

from test_gpu_masks import masked_attn_case
from test_gpu_parity_small import run_layer_case

pytestmark = pytest.mark.gpu

H64 = dict(dtype="bf16", hidden=256, n_q_heads=4, n_kv_heads=2, head_dim=64, mlp_width=512, vocab=1024)


@pytest.mark.parametrize("s,c,window,kv_first", [
    (0, 1, 0, 0), (0, 64, 0, 0), (63, 2, 0, 0), (300, 177, 100, 0), (1000, 256, 300, 0), (256, 200, 0, 70), (0, 300, 0, 130),
    (500, 130, 64, 520), (513, 255, 1, 0)])
def test_masked_attention_bf16_dh64(s, c, window, kv_first):
    before = sb.streambp_generic_launches()
    masked_attn_case("bf16", 6, 2, 64, s, c, window, kv_first)
    assert sb.streambp_generic_launches() == before


# 160 workgroups of 256 queries fill the chip better than 288 of 128: the form without the split over keys, masked and ragged
@pytest.mark.parametrize("dh,window,kv_first", [(64, 0, 0), (64, 300, 70), (128, 0, 0), (128, 300, 70)])
def test_masked_attention_bf16_whole_query_tiles(dh, window, kv_first):
    masked_attn_case("bf16", 32, 2, dh, 200, 1100, window, kv_first)


@pytest.mark.parametrize("T,chunk,batch", [(333, 100, 2), (640, 256, 1)])
def test_layer_backward_bf16_dh64(T, chunk, batch):
    before = sb.streambp_generic_launches()
    run_layer_case(H64, T, chunk, batch=batch, seed=4)
    assert sb.streambp_generic_launches() == before


# one visible pair of keys, a short block, peaked rows, both forms of the forward at long prefixes, a window of two keys
@pytest.mark.parametrize("hq,hkv,s,c,window,kv_first,q_scale", [
    (4, 4, 0, 2, 0, 0, 1.0), (4, 2, 0, 33, 0, 0, 1.0), (16, 4, 0, 512, 0, 0, 4.0), (8, 2, 2000, 300, 0, 0, 1.0), (8, 2, 2000, 300, 500, 70, 2.0),
    (32, 2, 200, 1100, 0, 0, 1.0), (8, 8, 100, 64, 2, 0, 3.0), (8, 2, 8000, 200, 0, 0, 0.5)])
def test_dh64_is_as_close_to_fp64_as_the_fp32_kernels(hq, hkv, s, c, window, kv_first, q_scale):
    """The shape-agnostic kernels hold scores, probabilities and statistics in fp32.  Log-sum-exp and dv leave as fp32: two kernels that
    round them at the same places differ by the order of their sums, a quarter of the error at most here (two bf16 terms in place of a
    probability: 2 to 14 times the error).  o and dq are rounded to bf16 and dk follows o through delta: the error of those
    roundings, equal in both, covers the rest."""
    gen = torch.Generator(device="cuda").manual_seed(hq * 1000 + s + c)
    n = s + c
    r = lambda rows, heads: torch.randn((rows, heads, 64), generator=gen, device="cuda")
    q, k, v, d_o = (r(c, hq) * q_scale).bfloat16(), r(n, hkv).bfloat16(), r(n, hkv).bfloat16(), r(c, hq).bfloat16()
    key, pos = torch.arange(n, device="cuda"), torch.arange(c, device="cuda")[:, None] + s
    seen = (key <= pos) & (key >= kv_first)
    if window:
        seen &= key > pos - window
    ref = dict(o=[], lse=[], dq=[], dk=[0.0] * hkv, dv=[0.0] * hkv)
    for h in range(hq):
        g = h // (hq // hkv)
        Q, K, V, DO = q[:, h].double(), k[:, g].double(), v[:, g].double(), d_o[:, h].double()
        S = (Q @ K.t() * 0.125).masked_fill(~seen, -float("inf"))
        lse = torch.logsumexp(S, 1)
        P, DP = torch.exp(S - lse[:, None]), DO @ V.t()
        DS = P * (DP - (P * DP).sum(1, keepdim=True)) * 0.125
        ref["o"].append(P @ V); ref["lse"].append(lse); ref["dq"].append(DS @ K)
        ref["dk"][g] = ref["dk"][g] + DS.t() @ Q
        ref["dv"][g] = ref["dv"][g] + P.t() @ DO
    ref = {n_: torch.stack(t, 0 if n_ == "lse" else 1) for n_, t in ref.items()}
    cfg = sb.attn_cfg(sb.SBP_BF16, hq, hkv, 64, s, c, 0.125, window, kv_first)
    err = {}
    try:
        for generic in (True, False):
            sb.debug_force_generic(attn=generic)
            o, lse = sb.streambp_attn_chunk_forward(cfg, q, k, v)
            dq, dk, dv = sb.streambp_attn_chunk_backward(cfg, q, k, v, o, lse, d_o)
            got = dict(o=o, lse=lse, dq=dq, dk=dk, dv=dv)
            err[generic] = {n_: float((got[n_].double() - t).norm() / t.norm()) for n_, t in ref.items()}
    finally:
        sb.debug_force_generic()
    for n_, factor in dict(o=1.01, dq=1.01, dk=1.01, lse=1.25, dv=1.25).items():
        assert err[False][n_] <= factor * err[True][n_] + 2.0 ** -26, (n_, err)
