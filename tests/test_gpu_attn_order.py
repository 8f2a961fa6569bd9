"""A short chunk behind a long prefix: the workgroups of dQ before those of dK/dV in one launch, with and without slices of dK/dV, halves of its columns,
windows and padding, as many key blocks as there are, against the fp64 oracle; and the sizes next to them, where dQ comes last."""
import pytest
import torch

from paper_2506_03077_amd import binding as sb
from test_gpu_masks import masked_attn_case

pytestmark = pytest.mark.gpu


# hq, hkv, start, queries, window, kv_first
@pytest.mark.parametrize("hq,hkv,s,c,window,kv_first", [
    (12, 2, 2000, 130, 0, 0),              # slices
    (28, 4, 3001, 255, 0, 700),            # a ragged chunk behind padding
    (64, 32, 7000, 130, 0, 0),             # more workgroups than one launch takes with dQ last
    (32, 32, 4000, 3, 0, 3990),            # only the last key block
    (8, 4, 3000, 140, 1300, 1800),         # a window: many key steps of dQ, few of dK/dV
    (8, 4, 3000, 600, 700, 0),             # ... and about as many of both
    (24, 3, 2500, 1025, 0, 0),             # 216 workgroups of dQ: last
])
@pytest.mark.parametrize("dh", [128, 64])
def test_a_short_chunk_behind_a_prefix(dh, hq, hkv, s, c, window, kv_first):
    q, k, v, d_o, ac, o, lse, *whole, _ = masked_attn_case("bf16", hq, hkv, dh, s, c, window, kv_first)
    if c < 200:      # (the built-in scratch holds no slices of dK/dV: one after the other, or in halves of the columns)
        dq, dk, dv = torch.empty_like(q), torch.zeros_like(whole[1]), torch.zeros_like(whole[2])
        assert all(torch.equal(a, b) for a, b in zip(whole, sb.streambp_attn_chunk_backward_noalloc(ac, q, k, v, o, lse, d_o, dq, dk, dv)))
