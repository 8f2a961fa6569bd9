"""The order of the query tiles where forward and dQ are more than one round of 256 workgroups: heads that do and do not divide among the eight XCDs, with
sequences, against the fp64 oracle."""
import pytest

from layer_plan_cases import MORE_THAN_A_ROUND
from test_gpu_attn_sequences import test_sequences_share_the_attention_launches as sequences
from test_gpu_masks import masked_attn_case

pytestmark = pytest.mark.gpu


# tiles of 128 or 256 queries times heads: 301 = 7 x 43, 258 = 6 x 43, 272 = 2 x 136, 264 = 8 x 33
@pytest.mark.parametrize("hq,hkv,s,c,window,kv_first", [(43, 43, 0, 800, 0, 0), (86, 43, 10, 300, 100, 0), (136, 8, 0, 200, 0, 30), (33, 11, 5, 900, 0, 0)])
@pytest.mark.parametrize("dh", [64, 128])
def test_more_than_a_round(hq, hkv, s, c, window, kv_first, dh):
    masked_attn_case("bf16", hq, hkv, dh, s, c, window, kv_first)


def test_sequences():
    sequences(MORE_THAN_A_ROUND)
