"""Which query tiles, launches and order the sizes of an attention call pick (csrc/attn_plan.h), on the CPU: the calls of the GPU tests are dealt as these say."""
import json
import os
import re
import shutil
import subprocess

import pytest

import test_gpu_attn_order
import test_gpu_attn_tile_choice as tile_choice
import test_gpu_generic_attn_one_launch as narrow

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "tests", "host_sanitize")
CSRC = os.path.join(ROOT, "paper_2506_03077_amd", "csrc")


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    out = str(tmp_path_factory.mktemp("attn_plans") / "attn_plans")
    p = subprocess.run([gxx, "-std=c++17", "-O1", "-I", SRC, "-I", CSRC, os.path.join(SRC, "attn_plans.cpp"), "-o", out], capture_output=True, text=True)
    assert p.returncode == 0, p.stderr[-4000:]
    with open(os.path.join(CSRC, "attn_mfma.hip")) as f:
        text = f.read()
    most = [int(re.search(rf"{n} = (\d+);", text).group(1)) for n in ("MERGED_MAX", "MERGED_MAX_PREFIX")]

    def run(hq, hkv, start, queries, window=0, kv_first=0, dh=128, sequences=1, room=1):
        line = " ".join(map(str, (dh, hq, hkv, start, queries, window, kv_first, sequences, room, *most)))
        p = subprocess.run([out], input=line, capture_output=True, text=True, timeout=60)
        assert p.returncode == 0, p.stderr[-2000:]
        return json.loads(p.stdout)
    return run


# A window's dQ tile sees the window and its own keys, however long the chunk is: the key blocks, which as many queries see, are no shorter.
@pytest.mark.parametrize("hq,hkv,start,queries,window", [(8, 8, 2730, 2184, 333), (8, 8, 0, 2340, 165), (12, 2, 30159, 1034, 351), (40, 8, 9284, 997, 64)])
@pytest.mark.parametrize("dh", [128, 64])
def test_a_long_chunk_under_a_window_does_not_begin_with_dq(plan, dh, hq, hkv, start, queries, window):
    p = plan(hq, hkv, start, queries, window, dh=dh)
    assert p["one_launch"] and p["n_dq"] <= 192 and not p["dq_first"]


def test_a_short_chunk_behind_many_keys_begins_with_dq(plan):
    for args in ((12, 2, 2000, 130), (64, 32, 7000, 130), (16, 16, 24442, 81), (64, 8, 6926, 129, 697), (32, 8, 8000, 640)):
        p = plan(*args)
        assert p["one_launch"] and p["dq_first"], args
    assert not plan(28, 4, 30720, 2048)["dq_first"]        # 224 workgroups of dQ


def test_neighbouring_prefixes_take_the_same_launches(plan):
    """Whole rounds of dK/dV are no case of their own: a prefix that is one key block shorter or longer is dealt alike."""
    for hq, hkv, start, queries in ((28, 4, 30720, 2048), (40, 8, 15754, 572), (40, 8, 7120, 1068), (28, 4, 14336, 2048)):
        got = [plan(hq, hkv, start + d, queries) for d in (-128, 0, 128)]
        assert any(p["n_dkv"] % 256 == 0 for p in got) and all(p["one_launch"] for p in got), got


def test_key_blocks_lie_side_by_side_where_there_is_nothing_to_even_out(plan):
    assert plan(16, 4, 1183, 117)["side_by_side"]                          # a CU for each workgroup
    assert plan(28, 4, 28672, 4096)["side_by_side"]                        # 32 of 256 blocks are the chunk's own
    assert not plan(28, 4, 28544, 4224)["side_by_side"]                    # ... one more
    assert not plan(28, 4, 0, 2048)["side_by_side"]
    assert not plan(64, 32, 7000, 130)["side_by_side"]                     # dQ first


def test_forward_tiles_of_64_wide_heads(plan):
    """Half tiles cost these heads less than the wider ones: whole tiles only where they leave few CUs idle."""
    for args in ((32, 8, 0, 2398, 2509), (28, 4, 9300, 3302, 124), (28, 4, 1852, 2767)):
        assert plan(*args, dh=64)["forward_halves"], args
    assert plan(32, 8, 0, 2398, 2509)["forward_halves"] == 0
    assert not plan(32, 8, 927, 3613, dh=64)["forward_halves"]


def _parameters(test, names):
    """The values a GPU test is parametrised over."""
    return next(m.args[1] for m in test.pytestmark if m.name == "parametrize" and m.args[0] == names)


def test_calls_of_the_tile_tests(plan):
    for args in tile_choice.WHOLE:
        p = plan(*args)
        assert not p["halves"] and not p["forward_halves"], args
        assert not plan(*args, dh=64)["halves"], args
    for args in tile_choice.HALF:
        assert all(p["halves"] and p["forward_halves"] for p in (plan(*args), plan(*args, dh=64))), args
    first, last = [plan(*a, dh=64) for a in tile_choice.DQ_FIRST], [plan(*a, dh=64) for a in tile_choice.DKV_FIRST]
    assert all(p["one_launch"] and p["dq_first"] for p in first)
    assert first[0]["n_dkv"] > 1024 and first[1]["n_dkv"] % 256 == 0
    assert not any(p["dq_first"] for p in last)
    assert last[0]["one_launch"] and last[0]["n_dkv"] > 1024 and not last[1]["one_launch"]


def test_calls_of_the_order_tests(plan):
    calls = _parameters(test_gpu_attn_order.test_a_short_chunk_behind_a_prefix, "hq,hkv,s,c,window,kv_first")
    got = {c: [plan(*c, dh=dh) for dh in (128, 64)] for c in calls}
    assert all(p["one_launch"] for ps in got.values() for p in ps)
    last = {c for c, ps in got.items() if not all(p["dq_first"] for p in ps)}
    assert last == {(32, 32, 4000, 3, 0, 3990), (24, 3, 2500, 1025, 0, 0)}
    assert any(p["parts"] and p["dq_first"] for ps in got.values() for p in ps)
    assert any(p["n_dkv"] + p["n_dq"] > 1536 and p["dq_first"] for ps in got.values() for p in ps)
    in_turn = [plan(*c, room=0) for c in calls if c[3] < 200]
    assert any(p["in_turn"] for p in in_turn) and any(p["in_turn"] and p["dq_first"] for p in in_turn)


def test_calls_of_the_narrow_tests(plan):
    calls = _parameters(narrow.test_backward, "dtype,hq,hkv,dh,s,c,window,kv_first")
    got = [plan(hq, hkv, s, c, window, kv_first, dh=dh) for _, hq, hkv, dh, s, c, window, kv_first in calls]
    kinds = [(p["narrow_one_launch"], p["narrow_dq_first"]) for p in got]
    assert kinds == [(1, 0)] * 7 + [(1, 1)] * 4 + [(0, 1)], kinds
    assert got[10]["narrow_n"] > 1024 and not any(p["narrow_in_place"] for p in got)
