"""Query tiles of 128 or 256 and key blocks dealt to workgroups by their work: chunks on both sides of the rule, with prefixes, windows, padding and
ragged ends, as many workgroups as CUs and more, against the fp64 oracle."""
import pytest

from test_gpu_masks import masked_attn_case

pytestmark = pytest.mark.gpu

# hq, hkv, start, queries, window, kv_first
WHOLE = [(64, 2, 900, 1000, 0, 0),            # a round of whole tiles, all about as long
         (64, 2, 900, 1000, 300, 950),        # ... under a window, behind padding that ends inside the chunk
         (128, 4, 0, 500, 0, 33)]             # two rounds of short ones
HALF = [(28, 4, 0, 1100, 0, 0),               # causal from 0: the longest whole tile would be the launch
        (28, 4, 300, 777, 256, 310),
        (12, 12, 0, 640, 0, 5)]               # key blocks times heads not a multiple of the XCDs


@pytest.mark.parametrize("hq,hkv,s,c,window,kv_first", WHOLE + HALF)
@pytest.mark.parametrize("dh", [128, 64])
def test_both_sides_of_the_rule(dh, hq, hkv, s, c, window, kv_first):
    masked_attn_case("bf16", hq, hkv, dh, s, c, window, kv_first)


# A chunk behind a prefix, dQ's workgroups first in one launch: more than 1024 workgroups, whole rounds of dK/dV, neither
DQ_FIRST = [(64, 32, 4000, 200), (32, 16, 3965, 130), (32, 32, 2000, 500)]
# ... dK/dV's first, 208 workgroups of dQ behind them: more than 1024 workgroups in one launch, more than 1536 apart
DKV_FIRST = [(208, 26, 5000, 100), (208, 52, 5000, 100)]


@pytest.mark.parametrize("hq,hkv,s,c", DQ_FIRST + DKV_FIRST)
def test_backward_behind_a_prefix(hq, hkv, s, c):
    masked_attn_case("bf16", hq, hkv, 64, s, c, 0, 0)
