"""How a layer call deals its rows to passes and weight-gradient launches, seen from the host layer's calls (tests/host_sanitize/plans.cpp, CPU only)."""
import itertools
import json
import os
import re
import shutil
import subprocess

import pytest

from layer_plan_cases import GROUPS, MORE_THAN_A_ROUND, PARTS, PASSES, SEQUENCES

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "tests", "host_sanitize")
CSRC = os.path.join(ROOT, "paper_2506_03077_amd", "csrc")


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    out = str(tmp_path_factory.mktemp("plans") / "plans")
    p = subprocess.run([gxx, "-std=c++17", "-O1", "-I", SRC, "-I", CSRC, "-x", "c++", os.path.join(CSRC, "api.hip"), os.path.join(SRC, "stub_launch.cpp"),
                        os.path.join(SRC, "plans.cpp"), "-o", out], capture_output=True, text=True)
    assert p.returncode == 0, p.stderr[-4000:]

    def run(configs):
        lines = []
        for c in configs:
            c = dict(dict(dtype="bf16", grad="f32", B=1, group=0, window=0, first=None), **c)
            lines.append([int(c["dtype"] == "bf16"), int(c["grad"] == "bf16"), c["B"], c["T"], c["chunk"], c["group"], c["hidden"], c["n_q_heads"], c["n_kv_heads"],
                          c["head_dim"], c["mlp_width"], c["window"], int(c["first"] is not None), *(c["first"] or [])])
        p = subprocess.run([out], input="\n".join(" ".join(map(str, li)) for li in lines), capture_output=True, text=True, timeout=600)
        assert p.returncode == 0, (p.stdout[-500:], p.stderr[-2000:])
        got = [json.loads(li) for li in p.stdout.splitlines()]
        assert len(got) == len(configs)
        return got
    return run


def _w(d, hq, hkv, dh, F):
    return dict(hidden=d, n_q_heads=hq, n_kv_heads=hkv, head_dim=dh, mlp_width=F)


WIDTHS = [_w(4096, 32, 8, 128, 14336), _w(2048, 16, 4, 128, 5632), _w(1024, 16, 4, 64, 2816), _w(256, 4, 2, 128, 64), _w(72, 6, 2, 24, 172)]
SWEEP = [dict(w, B=B, T=T, chunk=chunk, group=group) for w, (B, T), chunk, group in
         itertools.product(WIDTHS, [(1, 2048), (1, 8192), (1, 32768), (1, 5001), (4, 640), (3, 1300), (33, 20)], [64, 256, 1000, 1024, 4096], [0, 1, 3000])]


def _chunks(c):
    """Chunks of a call and chunks of a weight-gradient group, as the configuration says."""
    cm = min(c["chunk"], c["T"])
    return c["B"] * -(-c["T"] // cm), max(1, min(8, (c["group"] or 8192) // cm))


def test_bf16_gradients_are_rounded_no_more_often_than_chunk_by_chunk(plans):
    """A bf16 weight gradient is read, added to and rounded once per launch (once per pass where the launch cannot take several): fewer, larger passes
    must not come with more launches than groups of dw_group_rows rows make, and never with more passes than there are chunks."""
    configs = [dict(c, grad="bf16") for c in SWEEP]
    for c, got in zip(configs, plans(configs)):
        chunks, group = _chunks(c)
        assert len(got["dw"]) <= -(-chunks // group) and sum(map(len, got["dw"])) <= chunks, (c, got["dw"])


@pytest.mark.parametrize("grad", ["f32", "bf16"])
def test_every_row_is_in_one_pass(plans, grad):
    configs = [dict(c, grad=grad) for c in SWEEP]
    for c, got in zip(configs, plans(configs)):
        rows = sorted(r for launch in got["dw"] for r in launch)
        assert rows[0][0] == 0 and all(a + n == b for (a, n), (b, _) in zip(rows, rows[1:])) and sum(rows[-1]) == c["B"] * c["T"], (c, rows)
        for calls in (got["backward"], got["forward"]):
            assert sum(n * q for n, _, q, _, _ in calls) == c["B"] * c["T"], (c, calls)
            assert all(n == 1 or (s == 0 and q == c["T"] and n <= 32) for n, s, q, _, _ in calls), (c, calls)


def test_calls_that_share_attention_launches_are_dealt_as_their_tests_say(plans):
    """... and their sizes pick the kernels that the tests name: one launch for dQ and dK/dV up to MERGED_MAX workgroups, either query tile counted."""
    with open(os.path.join(CSRC, "attn_mfma.hip")) as f:
        merged_max = int(re.search(r"MERGED_MAX = (\d+);", f.read()).group(1))
    calls = SEQUENCES + [MORE_THAN_A_ROUND]
    for c, got in zip(calls, plans([dict(c["cfg"], B=c["B"], T=c["T"], chunk=c["T"], first=c["first"]) for c in calls])):
        assert [a[:3] for a in got["backward"]] == [[n, 0, c["T"]] for n in c["passes"]] and {a[3] for a in got["backward"]} == {c["slices"]}, (c, got)
        assert all(side_by_side == int(c["slices"] > 1) for *_, side_by_side in got["backward"]), (c, got)
        n, T = max(c["passes"]), c["T"]
        tiles = [-(-T // q) * c["cfg"]["n_q_heads"] * n for q in (256, 128)]
        hidden = min(c["first"]) // 128 if c["first"] else 0
        dkv = (-(-T // 128) - hidden) * c["cfg"]["n_kv_heads"] * n * c["slices"]
        assert c is not MORE_THAN_A_ROUND or min(tiles) > 256
        assert dkv + min(tiles) > merged_max if c["separate"] else dkv + max(tiles) <= merged_max, (c, dkv, tiles)


def test_passes_of_a_layer_are_dealt_as_their_test_says(plans):
    configs = [dict(cfg, B=B, T=T, chunk=chunk, group=group, window=window, first=first) for cfg, B, T, chunk, group, window, first, _, _ in PASSES]
    for (*_, dw, forward), got in zip(PASSES, plans(configs)):
        assert got["dw"] == dw and [a[:3] for a in got["forward"]] == forward, got


def test_groups_of_passes_and_parts_of_a_sequence_are_dealt_as_their_tests_say(plans):
    configs = [dict(cfg, B=B, T=T, chunk=chunk, group=group, grad="bf16") for cfg, B, T, chunk, group, _ in GROUPS]
    for (*_, sizes), got in zip(GROUPS, plans(configs)):
        assert [len(launch) for launch in got["dw"]] == sizes, got
    for p, got in zip(PARTS.values(), plans([dict(p["cfg"], B=1, T=p["T"], chunk=p["chunk"], group=p["group"]) for p in PARTS.values()])):
        assert [rows for _, _, rows, *_ in reversed(got["backward"])] == p["backward"], (p, got)
        assert not p["forward"] or [rows for _, _, rows, *_ in got["forward"]] == p["forward"], (p, got)
