"""The task engine counts a tile as done only after every wavefront of the
workgroup has run its part of it (CPU only).

What a tile stores cannot show this: a task that shares no data with another
has no reader before the engine ends, and its stamps are drawn by the one
wavefront that finishes it. So the order is checked in the flow graph of the
kernel, as compiled from its source to the compiler's intermediate form: on no
path does a store or count of a tile's data reach one of the engine's counters
(tiles done, in-degrees, work reserved, the next claim) without a workgroup
barrier in between.
"""
import os
import re
import subprocess

import pytest

from paper_2209_10643_amd import build as B

pytestmark = pytest.mark.skipif(not os.path.exists(B.HIPCC), reason="needs hipcc")

# The data's addresses come from task descriptors (generic pointers), the
# counters' from the kernel's argument (global pointers).
DATA = re.compile(r"raw\.ptr\.buffer\.store|store (float|atomic i32) %\S+, ptr %|atomicrmw add ptr %")
COUNTER = re.compile(r"atomicrmw add ptr addrspace\(1\) %\S+, i32")
BARRIER = "@llvm.amdgcn.s.barrier("


def kernel_blocks(tmp_path):
    """Basic blocks of the engine kernel: label -> (instructions, labels it goes on to)."""
    out = str(tmp_path / "task_engine.ll")
    subprocess.run([B.HIPCC, *B.FLAGS, "--offload-device-only", "-emit-llvm", "-S",
                    os.path.join(B.CSRC, "task_engine.hip"), "-o", out], check=True, capture_output=True)
    body = re.search(r"^define [^\n]*k_engineENS_7EngineDE[^\n]*\{\n(.*?)^\}", open(out).read(), re.S | re.M).group(1)
    blocks, name = {}, None
    for line in body.split("\n"):
        label = re.match(r"([\w.]+):", line)
        if label or name is None:
            name = label.group(1) if label else "entry"
            blocks[name] = ([], [])
            if label:
                continue
        code, out_to = blocks[name]
        code.append(line.strip())
        # a terminator's labels, also on the lines of a switch's table
        out_to += re.findall(r"label %([\w.]+)", line)
    return blocks


def test_every_tile_passes_a_barrier_before_it_counts(tmp_path):
    blocks = kernel_blocks(tmp_path)
    every = [c for code, _ in blocks.values() for c in code]
    assert sum(bool(DATA.search(c)) for c in every) > 20 and sum(bool(COUNTER.search(c)) for c in every) >= 4
    assert any(BARRIER in c for c in every)
    seen, todo = set(), []

    def walk(name, first, after_data):
        for c in blocks[name][0][first:]:
            if BARRIER in c:
                after_data = False
            elif after_data:
                assert not COUNTER.search(c), f"block {name}: reached with no barrier after a tile's stores: {c[:80]}"
            if DATA.search(c):
                after_data = True
        if after_data:
            todo.extend(b for b in blocks[name][1] if b not in seen)

    for name in blocks:
        walk(name, 0, False)
    while todo:
        name = todo.pop()
        if name not in seen:
            seen.add(name)
            walk(name, 0, True)
