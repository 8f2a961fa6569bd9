"""dK/dV without room for the sums of a key block's shares, at both sides of the rule that decides how they are taken one after the other: the
same bits as with room (the sums and their order are the same), also where a share has no step."""
import pytest
import torch

from paper_2506_03077_amd import binding as sb

pytestmark = pytest.mark.gpu

# hq, hkv, dh, start, queries, window, kv_first
SHAPES = [(64, 8, 128, 1400, 100, 0, 0),      # 12 key blocks x 8: the last that two workgroups each share
          (64, 8, 128, 1500, 100, 0, 0),      # 13 x 8: one workgroup each, share after share
          (8, 1, 128, 0, 64, 0, 0),           # one key block, one query tile
          (8, 1, 128, 200, 260, 60, 3),       # key blocks with fewer steps than shares, a window and padding
          (4, 4, 64, 0, 300, 0, 0), (16, 2, 64, 1000, 33, 0, 0)]


@pytest.mark.parametrize("hq,hkv,dh,s,c,window,kv_first", SHAPES)
def test_shares_one_after_the_other_give_the_same_bits(hq, hkv, dh, s, c, window, kv_first):
    gen = torch.Generator(device="cuda").manual_seed(7 + s + c)
    r = lambda rows, heads: torch.randn((rows, heads, dh), generator=gen, device="cuda").bfloat16()
    q, k, v, d_o = r(c, hq), r(s + c, hkv), r(s + c, hkv), r(c, hq)
    ac = sb.attn_cfg(sb.SBP_BF16, hq, hkv, dh, s, c, dh ** -0.5, window, kv_first)
    need, least = sb.streambp_attn_workspace_bytes(ac), -(-2 * c * hq * 4 // 256) * 256
    assert need > least, "a shape whose queries are not cut shows nothing"
    o, lse = sb.streambp_attn_chunk_forward(ac, q, k, v)
    start = [torch.randn((s + c, hkv, dh), generator=gen, device="cuda") for _ in range(2)]      # dk, dv are added to
    call = lambda room: sb.streambp_attn_chunk_backward(ac, q, k, v, o, lse, d_o, dk=start[0].clone(), dv=start[1].clone(),
                                                        workspace=torch.full((room,), 0xFF, dtype=torch.uint8, device="cuda"))
    whole = call(need)
    dq, dk, dv = torch.full_like(q, float("nan")), start[0].clone(), start[1].clone()
    assert all(torch.equal(a, b) for a, b in zip(whole, call(least)))
    assert all(torch.equal(a, b) for a, b in zip(whole, sb.streambp_attn_chunk_backward_noalloc(ac, q, k, v, o, lse, d_o, dq, dk, dv)))
