"""Hand-overs between workgroups, checked in the gfx950 assembly of the
kernels: where a workgroup counts itself done so that others read its stores,
every wavefront has waited for its own stores before the barrier that precedes
the count.  (A workgroup-scope fence and a barrier order stores within one CU
only; the CPU build's fences are sequentially consistent and cannot show a
missing wait.)"""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "paper_2606_24531_amd", "csrc", "kernels.hip")

# kernel, the returning atomic adds that publish a workgroup's stores
CASES = [("k_chain", r"(global|flat)_atomic_add v"), ("k_persist", r"(global|flat)_atomic_add_x2 v")]


@pytest.fixture(scope="module")
def asm(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("isa") / "kernels.s")
    subprocess.check_call(["hipcc", "-S", "--offload-device-only", "-O3", "-std=c++17", "--offload-arch=gfx950",
                           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-x", "hip", SRC, "-o", out],
                          stderr=subprocess.DEVNULL)
    with open(out) as f:
        return f.read()


def _blocks(asm, kernel):
    """The kernel's basic blocks in layout order: (label, instructions)."""
    m = re.search(r"^(_Z\w*%s\w*):.*?^\.Lfunc_end\d+:" % kernel, asm, re.M | re.S)
    blocks, cur = [], ("entry", [])
    for line in m.group(0).split("\n")[1:]:
        line = line.split(";")[0].strip()
        label = re.match(r"(\.LBB\w+):", line)
        if label:
            blocks.append(cur)
            cur = (label.group(1), [])
        elif line and not line.startswith("."):
            cur[1].append(line)
            if re.match(r"s_(c?branch\w*|endpgm)", line):  # what follows is a block of its own
                blocks.append(cur)
                cur = ("", [])
    return blocks + [cur]


def _unwaited(blocks, publish):
    """(published adds seen, those that a path reaches whose last barrier was
    passed with a store unwaited for).  State of a path: a store issued since
    the last full wait; the same at its last barrier."""
    at = {b[0]: i for i, b in enumerate(blocks) if b[0]}
    state = [None] * len(blocks)
    state[0] = (False, False)
    todo, seen, bad = [0], set(), set()
    while todo:
        i = todo.pop()
        dirty, barrier = state[i]
        nxt = [i + 1]
        for k, ins in enumerate(blocks[i][1]):
            if re.match(r"(global|flat|buffer)_store", ins):
                dirty = True
            elif ins.startswith("s_waitcnt") and "vmcnt(0)" in ins:
                dirty = False
            elif ins.startswith("s_barrier"):
                barrier = dirty
            elif re.match(publish, ins) and re.search(r"\bsc0\b", ins):
                seen.add((i, k))
                if barrier:
                    bad.add((i, k))
            elif ins.startswith("s_branch"):
                nxt = [at[ins.split()[1]]]
            elif ins.startswith("s_cbranch"):
                nxt.append(at[ins.split()[1]])
            elif ins.startswith("s_endpgm"):
                nxt = []
        for j in nxt:
            if j >= len(blocks):
                continue
            old = state[j] or (False, False)
            new = (old[0] or dirty, old[1] or barrier)
            if state[j] is None or new != old:
                state[j] = new
                todo.append(j)
    return seen, bad


@pytest.mark.parametrize("kernel,publish", CASES, ids=[c[0] for c in CASES])
def test_stores_are_waited_for_before_they_are_counted(asm, kernel, publish):
    blocks = _blocks(asm, kernel)
    stores = sum(bool(re.match(r"(global|flat|buffer)_store", i)) for b in blocks for i in b[1])
    seen, bad = _unwaited(blocks, publish)
    assert stores and seen
    assert not bad, [blocks[i][1][k] for i, k in bad]
