"""dQ in slots: no key tile, one, few and many, at every remainder of the four LDS stages, with ragged first and last tiles, in both forms (256
queries per workgroup, tiles of 64 keys; 128 queries, two groups on the even / odd tiles of 32 keys), against the fp64 oracle."""
import pytest

from test_gpu_masks import masked_attn_case

pytestmark = pytest.mark.gpu

# start, queries, window, kv_first: 1 to 6 tiles of 32 or 64 keys and a remainder, windows and padding that begin inside a tile, queries without a key
RANGES = [(0, 1, 0, 0), (0, 31, 0, 0), (1, 33, 0, 0), (40, 64, 0, 0), (100, 65, 0, 0), (129, 96, 0, 0), (255, 130, 0, 0), (97, 40, 33, 0),
          (300, 70, 64, 0), (70, 60, 0, 200), (64, 90, 0, 97), (10, 257, 40, 30)]


@pytest.mark.parametrize("s,c,window,kv_first", RANGES)
@pytest.mark.parametrize("dh", [128, 64])
def test_few_tiles(dh, s, c, window, kv_first):
    masked_attn_case("bf16", 4, 2, dh, s, c, window, kv_first)      # few workgroups: 128 queries each


@pytest.mark.parametrize("s,c,window,kv_first", [(0, 300, 0, 0), (190, 257, 0, 0), (61, 256, 50, 0), (33, 200, 0, 100)])
@pytest.mark.parametrize("dh", [128, 64])
def test_whole_query_tiles(dh, s, c, window, kv_first):
    """Enough heads that 256-query workgroups fill the chip."""
    masked_attn_case("bf16", 256 if c <= 256 else 128, 64, dh, s, c, window, kv_first)
