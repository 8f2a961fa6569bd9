"""Layer calls of the tests of passes, and how their rows are dealt: test_layer_plans.py reads the passes off the host layer on the CPU,
the GPU tests that import from here run them."""
from paper_2506_03077_amd import synth


def _seq(hq, hkv, dh, B, T, first, passes, slices, separate=False, window=0):
    """One chunk as long as a sequence.  passes: sequences of each pass of the backward; slices: workgroups that share a key block of dK/dV;
    separate: dQ and dK/dV have launches of their own."""
    return dict(cfg=dict(dtype="bf16", hidden=256, n_q_heads=hq, n_kv_heads=hkv, head_dim=dh, mlp_width=512, window=window), B=B, T=T, first=first,
                passes=passes, slices=slices, separate=separate)


SEQUENCES = [
    _seq(4, 2, 128, 3, 300, [130, 200, 299], [3], 5),              # the first key block hidden by all, the second by one
    _seq(4, 2, 64, 4, 257, [0, 150, 256, 257], [4], 5),            # a sequence without a visible key
    _seq(8, 2, 128, 4, 400, None, [4], 5, window=100),
    _seq(4, 4, 64, 5, 130, [0, 1, 2, 64, 129], [5], 1, window=33),
    _seq(4, 2, 128, 33, 20, list(range(20)) + [0] * 13, [4] * 8 + [1], 1),
    _seq(32, 8, 64, 32, 128, None, [4] * 8, 4),                    # many heads, still one launch of the backward
    _seq(20, 4, 64, 7, 260, [0, 3, 0, 130, 259, 1, 64], [4, 3], 5),
    _seq(32, 16, 64, 3, 1300, [0, 130, 1299], [3], 1, True),
    _seq(32, 16, 128, 3, 1300, [0, 130, 1299], [3], 1, True),
    _seq(32, 2, 64, 3, 1300, None, [3], 7, True),                  # ... and sums of parts
]
# 90 heads of all sequences, which do not divide among eight XCDs; more query tiles than a round of 256 workgroups, of 256 queries or of 128
MORE_THAN_A_ROUND = _seq(30, 6, 64, 3, 520, [0, 130, 519], [3], 2)

_MID = dict(dtype="bf16", hidden=256, n_q_heads=4, n_kv_heads=2, head_dim=128, mlp_width=512)
_NARROW = dict(dtype="bf16", hidden=256, n_q_heads=4, n_kv_heads=2, head_dim=64, mlp_width=64)      # an MLP that has no room for the rows of the K/V pass
_TINY = synth.CONFIGS["tiny"]


def _one(*rows):      # a weight-gradient launch a pass
    return [[r] for r in rows]


# bf16 weight gradients.  Config, batch, tokens, chunk, dw_group_rows; passes of each weight-gradient launch
GROUPS = [
    (_MID, 1, 1100, 64, 256, [2, 2, 2, 2, 1]),          # parts of a sequence
    (_MID, 4, 300, 64, 0, [3, 3, 2]),                   # parts of several
    (_MID, 5, 130, 64, 256, [4, 4, 2]),
    (_MID, 9, 100, 100, 512, [5, 4]),                   # whole sequences
    (dict(_MID, hidden=64, n_q_heads=8, n_kv_heads=8, head_dim=64, mlp_width=64), 4, 300, 256, 1, [8]),      # as many as a launch takes
]


def _part(cfg, T, chunk, group, backward, forward=None):
    """One sequence.  backward, forward: rows of its passes, in the order of the rows."""
    return dict(cfg=cfg, T=T, chunk=chunk, group=group, backward=backward, forward=forward)


_7B, _LLAMA = synth.CONFIGS["7b"], synth.CONFIGS["llama_layer"]
PARTS = {
    "7b benchmark": _part(_7B, 32768, 2048, 0, [4096] * 8),
    "7b small chunks": _part(_7B, 32768, 512, 0, [3328] * 9 + [2816]),
    "7b two in one launch": _part(_7B, 4608, 2048, 0, [2304] * 2),
    "7b ragged": _part(_7B, 4608, 512, 1, [659] * 6 + [654]),
    "7b whole": _part(_7B, 4608, 4608, 0, [4608]),
    "llama": _part(_LLAMA, 8192, 1024, 0, [4096] * 2),
    "llama ragged": _part(_LLAMA, 8192, 1000, 1, [1280] * 6 + [512]),
    "llama oracle": _part(_LLAMA, 2560, 1024, 1, [1280] * 2),
    "mid": _part(_MID, 640, 256, 1, [320] * 2),
    "mid small": _part(_MID, 640, 128, 1, [160] * 4, [320] * 2),
    "mid whole": _part(_MID, 640, 640, 1, [640]),
}

# config, batch, tokens, chunk, dw_group_rows, window, first; weight-gradient launches as [first row, rows] of their passes, in order; passes of the
# forward as [sequences, first row, rows]
PASSES = [
    (_MID, 5, 130, 64, 0, 0, [0, 129, 7, 130, 64],      # two sequences, two, one
     _one([0, 260], [260, 260], [520, 130]), [[3, 0, 130], [2, 0, 130]]),
    (_MID, 7, 100, 100, 250, 0, None,                   # one sequence a pass, two passes a weight-gradient launch, forward two a pass
     [[[0, 100], [100, 100]], [[200, 100], [300, 100]], [[400, 100], [500, 100]], [[600, 100]]], [[2, 0, 100]] * 3 + [[1, 0, 100]]),
    (_MID, 2, 333, 64, 1, 50, [0, 70],                  # four parts of a sequence, the last one shorter
     _one([252, 81], [168, 84], [84, 84], [0, 84], [585, 81], [501, 84], [417, 84], [333, 84]), [[1, 0, 167], [1, 167, 166]] * 2),
    (_NARROW, 3, 257, 64, 1, 0, None,
     _one([172, 85], [86, 86], [0, 86], [429, 85], [343, 86], [257, 86], [686, 85], [600, 86], [514, 86]), [[1, 0, 129], [1, 129, 128]] * 3),
    (_TINY, 5, 50, 40, 0, 16, [3, 0, 50, 49, 1],        # three sequences, two
     _one([0, 150], [150, 100]), [[5, 0, 50]]),
    (_TINY, 2, 200, 40, 1, 0, None,
     _one([150, 50], [100, 50], [50, 50], [0, 50], [350, 50], [300, 50], [250, 50], [200, 50]), [[1, 0, 100], [1, 100, 100]] * 2),
]
