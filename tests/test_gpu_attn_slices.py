"""dK/dV of short chunks: the queries of a key block cut into slices, a workgroup each where the workspace has room for their sums, one
after the other in one workgroup where it has not - the same bits either way - and against the fp64 oracle."""
import pytest
import torch

from paper_2506_03077_amd import binding as sb

from test_gpu_masks import masked_attn_case

pytestmark = pytest.mark.gpu

# hq, hkv, dh, start, queries, window, kv_first: one and many key blocks, ragged tiles, more slices than some blocks have steps, a window,
# blocks hidden by padding, 64-wide heads
SHAPES = [(8, 2, 128, 0, 130, 0, 0), (8, 2, 128, 1000, 77, 0, 0), (8, 2, 128, 300, 500, 0, 0), (4, 4, 128, 0, 700, 100, 0),
          (8, 2, 128, 640, 200, 0, 650), (8, 2, 64, 100, 333, 0, 5)]


@pytest.mark.parametrize("hq,hkv,dh,s,c,window,kv_first", SHAPES)
def test_slices_give_the_same_bits_with_and_without_room_for_their_sums(hq, hkv, dh, s, c, window, kv_first):
    gen = torch.Generator(device="cuda").manual_seed(s + c)
    r = lambda rows, heads: torch.randn((rows, heads, dh), generator=gen, device="cuda").bfloat16()
    q, k, v, d_o = r(c, hq), r(s + c, hkv), r(s + c, hkv), r(c, hq)
    ac = sb.attn_cfg(sb.SBP_BF16, hq, hkv, dh, s, c, dh ** -0.5, window, kv_first)
    need, least = sb.streambp_attn_workspace_bytes(ac), -(-2 * c * hq * 4 // 256) * 256
    assert need > least, "a shape whose queries are not cut shows nothing"
    o, lse = sb.streambp_attn_chunk_forward(ac, q, k, v)
    start = [torch.randn((s + c, hkv, dh), generator=gen, device="cuda") for _ in range(2)]      # dk, dv are added to
    got = []
    for room in (need, need - 1, least):
        ws = torch.full((room,), 0xFF, dtype=torch.uint8, device="cuda")
        got.append(sb.streambp_attn_chunk_backward(ac, q, k, v, o, lse, d_o, dk=start[0].clone(), dv=start[1].clone(), workspace=ws))
    for other in got[1:]:
        assert all(torch.equal(a, b) for a, b in zip(got[0], other))
    with pytest.raises(sb.StreamBPError):
        sb.streambp_attn_chunk_backward(ac, q, k, v, o, lse, d_o, workspace=torch.empty(least - 256, dtype=torch.uint8, device="cuda"))


@pytest.mark.parametrize("hq,hkv,dh,s,c,window,kv_first", SHAPES)
def test_slices_match_the_oracle(hq, hkv, dh, s, c, window, kv_first):
    masked_attn_case("bf16", hq, hkv, dh, s, c, window, kv_first)
