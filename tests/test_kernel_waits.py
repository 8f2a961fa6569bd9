"""Waits of the kernels that refill LDS by direct-to-LDS loads while other waves still read it, checked on the machine code that was
built: between such a refill and the last read of the buffer there is a barrier, and a barrier orders nothing that has not been
waited for.  Every path through a kernel's control flow is walked with the queue of LDS reads that no s_waitcnt has covered yet (LDS
operations of a wave complete in order), and the number of barriers each passes unwaited is bounded by what the kernel's schedule allows:

  GEMM       two: B0 is read in the last fetch slot of a K step and waited for in the first one of the next, two barriers later; the
             third barrier is the one after which the other wave group may refill that half
  attention  none: every fragment is consumed in the slot in which it is read"""
import glob
import os
import re
import shutil
import subprocess

import pytest

from paper_2506_03077_amd import build as B

OBJDUMP = os.environ.get("LLVM_OBJDUMP", "/opt/rocm/llvm/bin/llvm-objdump")
FORGET = 8          # barriers after which a read that is still unwaited is no longer followed


def kernels(lib, workdir):
    """{kernel name: [(address, mnemonic, operands, branch target)]} of the gfx950 code objects in the library."""
    copy = shutil.copy(lib, workdir)
    subprocess.run([OBJDUMP, "--offloading", copy], check=True, capture_output=True, cwd=workdir)
    out = {}
    for code in sorted(glob.glob(copy + "*gfx950")):
        if os.path.getsize(code) == 0:
            continue
        text = subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", "--no-show-raw-insn", code], check=True, capture_output=True, text=True).stdout
        body = None
        for line in text.splitlines():
            head = re.match(r"^[0-9a-f]+ <(.+)>:$", line)
            if head:
                body = out[head.group(1)] = []
                continue
            ins = re.match(r"^\s+(\S+)\s*(.*?)\s*// ([0-9A-F]+):", line)
            if ins and body is not None:
                addr, op, args, target = int(ins.group(3), 16), ins.group(1), ins.group(2), None
                if op.startswith(("s_cbranch", "s_branch")):
                    simm = int(args)
                    target = addr + 4 + 4 * (simm - 65536 if simm >= 32768 else simm)
                body.append((addr, op, args, target))
    return out


def barriers_passed_unwaited(code):
    """The largest number of barriers that any LDS read of the kernel passes before a wait covers it, over all paths."""
    index = {ins[0]: i for i, ins in enumerate(code)}

    def successors(i):
        _, op, _, target = code[i]
        if op == "s_endpgm":
            return []
        assert not op.startswith(("s_setpc", "s_swappc", "s_call")), "calls are not followed"
        if op.startswith("s_cbranch"):
            return [i + 1, index[target]]
        return [index[target]] if op == "s_branch" else [i + 1]

    targets = {index[ins[3]] for ins in code if ins[3] is not None}
    seen, work, worst = {(0, ())}, [(0, ())], 0
    while work:
        assert len(seen) < 400000, "too many states"
        i, queue = work.pop()          # queue: barriers passed by each uncovered LDS operation, oldest first (None: a write)
        while True:
            _, op, args, _ = code[i]
            if op.startswith("ds_read"):
                queue += (0,)
            elif op.startswith("ds_"):
                queue += (None,)
            elif op == "s_waitcnt":
                m = re.search(r"lgkmcnt\((\d+)\)", args)
                assert m or "cnt(" in args, f"unreadable wait: {args}"
                if m:
                    n = int(m.group(1))
                    queue = queue[len(queue) - n:] if 0 < n < len(queue) else (queue if n else ())
            elif op == "s_barrier":
                queue = tuple(a if a is None else a + 1 for a in queue if a is None or a < FORGET)
                worst = max([worst] + [a for a in queue if a is not None])
            nxt = successors(i)
            if len(nxt) == 1 and nxt[0] not in targets:
                i = nxt[0]
                continue
            for j in nxt:
                if (j, queue) not in seen:
                    seen.add((j, queue))
                    work.append((j, queue))
            break
    return worst


@pytest.fixture(scope="module")
def built(tmp_path_factory):
    if not os.path.exists(B.LIB):
        B.build(force=False, verbose=False)
    return kernels(B.LIB, str(tmp_path_factory.mktemp("code")))


def _named(built, parts):
    return {n: c for n, c in built.items() if any(p in n for p in parts)}


def test_no_gemm_refills_a_half_tile_that_may_still_be_read(built):
    found = _named(built, ("11gemm_mfma_k", "17gemm_mfma_group_k", "15gemm_mfma_seg_k"))
    assert len(found) >= 20
    worst = {n: barriers_passed_unwaited(c) for n, c in found.items()}
    assert max(worst.values()) <= 2, {n: w for n, w in worst.items() if w > 2}


def test_attention_kernels_consume_what_they_read_within_the_slot(built):
    found = _named(built, ("15attn_fwd_mfma_k", "18attn_bwd_dq_mfma_k", "19attn_bwd_dkv_mfma_k"))
    assert len(found) == 10
    worst = {n: barriers_passed_unwaited(c) for n, c in found.items()}
    assert max(worst.values()) == 0, {n: w for n, w in worst.items() if w}
