"""The shape-agnostic attention kernels' instances by head width, at both sides of the numbers of keys where heads of more than 64 elements change from four
waves per block to two (or sixteen waves), with ragged heads, a window and padding, against fp64; and hidden infinities in wide heads."""
import pytest

from test_gpu_attn_generic_edges import test_hidden_rows_reach_nothing as hidden_rows
from test_gpu_masks import masked_attn_case

pytestmark = pytest.mark.gpu

# heads of up to 128: 32 keys | 33; of up to 192: 128 | 129; wider: 256 | 257
CASES = [(33, 19, 21), (48, 0, 40), (49, 30, 17), (65, 0, 32), (65, 0, 33), (80, 20, 12), (96, 300, 33), (97, 20, 13), (127, 200, 9), (129, 100, 28),
         (129, 100, 29), (160, 0, 128), (160, 300, 45), (161, 96, 33), (192, 50, 78), (193, 200, 56), (193, 200, 57), (254, 0, 256), (255, 250, 33), (256, 240, 17)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("dh,s,c", CASES)
def test_instances(dtype, dh, s, c):
    masked_attn_case(dtype, 4, 2, dh, s, c, 0, 0)


@pytest.mark.parametrize("dtype,dh,s,c,window,kv_first", [("f32", 100, 90, 50, 37, 60), ("bf16", 130, 200, 40, 100, 170), ("f32", 256, 300, 31, 16, 0),
                                                          ("bf16", 190, 0, 40, 0, 35), ("f32", 256, 0, 20, 0, 30)])
def test_masks(dtype, dh, s, c, window, kv_first):
    masked_attn_case(dtype, 6, 2, dh, s, c, window, kv_first)


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("dtype,dh", [("f32", 250), ("bf16", 193), ("f32", 128)])
def test_hidden_rows_of_wide_heads_reach_nothing(dtype, dh, bad):
    hidden_rows(dtype, dh, bad)
