"""GPU parity of the MFMA attention kernels against the fp64 oracle: 64-wide heads (masked, ragged), whole 256-query tiles and the form
that splits the keys over the wave groups, a layer with 64-wide heads."""
import pytest

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
