"""Backward of the shape-agnostic attention for heads of up to 64 elements, dQ and dK/dV in one launch with either first and apart, against the fp64 oracle:
each number of 16-wide pieces, ragged heads, windows, padding, both storage types."""
import pytest
import torch

from paper_2506_03077_amd import binding as sb
from test_gpu_masks import masked_attn_case

pytestmark = pytest.mark.gpu


# hq, hkv, dh, start, queries, window, kv_first
@pytest.mark.parametrize("dtype,hq,hkv,dh,s,c,window,kv_first", [
    ("f32", 4, 2, 16, 0, 257, 0, 0), ("f32", 4, 4, 30, 0, 100, 33, 7), ("f32", 3, 1, 47, 70, 41, 0, 80), ("f32", 2, 2, 64, 0, 130, 0, 0),      # dK/dV first
    ("bf16", 4, 2, 8, 0, 33, 0, 0), ("bf16", 4, 2, 24, 3, 90, 20, 0), ("bf16", 2, 1, 40, 0, 300, 0, 299),
    ("f32", 2, 1, 16, 500, 17, 0, 0), ("f32", 8, 8, 33, 1100, 1, 0, 0), ("bf16", 2, 2, 48, 300, 50, 64, 260),                                   # dQ first
    ("f32", 16, 16, 20, 1100, 40, 0, 0),                                                                                                        # ... beyond 1024 workgroups
    ("f32", 16, 16, 16, 1000, 210, 0, 0),                                                                                                       # apart
])
def test_backward(dtype, hq, hkv, dh, s, c, window, kv_first):
    masked_attn_case(dtype, hq, hkv, dh, s, c, window, kv_first)


def test_dq_in_the_place_of_o():
    q, k, v, d_o, ac, o, lse, dq, dk, dv, _ = masked_attn_case("f32", 4, 2, 16, 30, 400, 0, 0)
    assert all(torch.equal(a, b) for a, b in zip((dq, dk, dv), sb.streambp_attn_chunk_backward(ac, q, k, v, o, lse, d_o, dq=o)))
