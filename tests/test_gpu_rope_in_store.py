"""RoPE of K in the store of its product (fp32): heads of 2 to 32 columns that divide a tile and others, one pass over whole sequences (q, K and V in one
launch) and row blocks, batches, a position offset, rows that end inside a tile, against the fp64 oracle."""
import pytest

from test_gpu_parity_small import run_layer_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dh", [2, 4, 8, 16, 32, 12, 24, 40])
@pytest.mark.parametrize("hq,hkv,T,chunk,batch,offset", [(4, 4, 70, 16, 1, 0), (4, 2, 45, 45, 3, 11)])
def test_layer(dh, hq, hkv, T, chunk, batch, offset):
    run_layer_case(dict(dtype="f32", hidden=48, n_q_heads=hq, n_kv_heads=hkv, head_dim=dh, mlp_width=100, vocab=64), T, chunk, batch, pos_offset=offset)
