"""Host-side check of the direct MoE kernel's waits, on the AMD assembly that hipcc makes of it: on every path
from an activation DMA into LDS to the next barrier stands an s_waitcnt that covers that DMA.

vmcnt counts the vector memory operations in flight, oldest first: after a DMA followed by n others,
``vmcnt(m)`` covers it if m <= n. The source counts on the weight and scale loads that follow a DMA to be
issued before its wait; a load that the compiler sinks past the wait would make the count too high. No test
here touches a GPU.
"""
import os
import re
import subprocess

import pytest

from paper_2607_19438_amd import build

SRC = os.path.join(build.CSRC, "moe_direct.hip")
VMEM = ("buffer_", "global_", "flat_", "scratch_")


def functions(text):
    name, body = None, []
    for line in text.splitlines():
        m = re.match(r"^(_Z\w+):", line)
        if m:
            name, body = m.group(1), []
        elif line.startswith(".Lfunc_end"):
            if name:
                yield name, body
            name = None
        elif name:
            body.append(line.split(";")[0].strip())


def blocks_of(body):
    blocks, order, cur = {"entry": []}, ["entry"], "entry"
    for line in body:
        m = re.match(r"^(\.LBB\w+):", line)
        if m:
            cur = m.group(1)
        elif not line or line.startswith("."):
            continue
        else:
            blocks[cur].append(line)
            if not line.startswith(("s_branch", "s_cbranch", "s_endpgm")):
                continue
            cur += "+"
        blocks[cur] = []
        order.append(cur)
    return blocks, dict(zip(order, order[1:]))


def walk(lines, state):
    """state: vector memory operations since the youngest DMA not yet covered by a wait, None without one.
    Returns the state at the end, the branch targets, whether the block falls through, and the barriers
    reached with a DMA uncovered."""
    targets, falls, late = [], True, []
    for line in lines:
        op = line.split()[0]
        assert op not in ("s_setpc_b64", "s_swappc_b64"), "calls are not followed"
        if op.startswith(VMEM):
            if re.search(r"\blds\b", line):
                state = 0
            elif state is not None:
                state += 1
        elif op == "s_waitcnt":
            m = re.search(r"vmcnt\((\d+)\)", line)
            if m and state is not None and int(m.group(1)) <= state:
                state = None
        elif op == "s_barrier" and state is not None:
            late.append(line)
        elif op.startswith("s_cbranch"):
            targets.append(line.split()[-1])
        elif op == "s_branch":
            targets, falls = targets + [line.split()[-1]], False
        elif op == "s_endpgm":
            falls = False
    return state, targets, falls, late


def late_barriers(body):
    """Barriers that some path reaches with a DMA uncovered."""
    blocks, following = blocks_of(body)
    at, work = {"entry": None}, ["entry"]
    while work:
        b = work.pop()
        state, targets, falls, _ = walk(blocks[b], at[b])
        for t in targets + ([following[b]] if falls and b in following else []):
            known = [s for s in (state, at.get(t)) if s is not None]
            worst = min(known) if known else None
            if t not in at or worst != at[t]:
                at[t] = worst
                work.append(t)
    return [x for b in at for x in walk(blocks[b], at[b])[3]]


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("asm") / "moe_direct.s")
    subprocess.run([build.HIPCC, *build.FLAGS, "-S", "--cuda-device-only", SRC, "-o", out], check=True,
                   stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    return open(out).read()


def test_every_dma_is_waited_for_before_its_barrier(assembly):
    kernels = dict(functions(assembly))
    assert len(kernels) >= 10
    for name, body in kernels.items():
        assert sum(bool(re.search(r"\blds\b", l)) for l in body if l.startswith("buffer_load")) > 0, name
        assert late_barriers(body) == [], name


def test_a_wait_one_too_loose_is_found(assembly):
    """Every counted wait of one kernel loosened by one: each of its loops reports it."""
    name, body = next((n, b) for n, b in functions(assembly) if "ILi1ELi1E" in n)
    loose = [re.sub(r"vmcnt\((\d+)\)", lambda m: f"vmcnt({int(m.group(1)) + 1})", l) for l in body]
    assert late_barriers(body) == []
    assert late_barriers(loose), name
