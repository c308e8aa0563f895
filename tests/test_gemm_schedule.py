"""The alternating GEMM tiles' LDS rule, checked on the kernels as built (host only).

In those tiles the two wavefronts of a SIMD swap roles at a bare workgroup barrier, and a
unit of the operand ring is loaded again four slots after one wavefront group read it, three
after the other.  The refill lands in LDS behind the compiler's back, so nothing but the
barriers orders it after the reads: every LDS read has to be in registers (a wait for
lgkmcnt(0)) after at most one barrier, on every path through the kernel, the prologue's
included.  The test follows all paths of the machine code that this tree built.
"""
import os
import re
import shutil
import subprocess

import pytest

from paper_2604_26294_amd.build import LIB

OBJDUMP = shutil.which("llvm-objdump", path="/opt/rocm/llvm/bin:" + os.environ.get("PATH", ""))
LABEL = re.compile(r"^([0-9a-f]+) <(\S+)>:$")
INSN = re.compile(r"^\s+(\S+)\s*(.*?)\s*//\s*([0-9A-F]+):")
TARGET = re.compile(r"<\S+?(?:\+0x([0-9a-f]+))?>\s*$")


def barriers_over_reads(insns, base):
    """Most barriers that an LDS read is still in flight over, on any path from the entry.
    insns: (address, mnemonic, operands, text) in order; branch targets are offsets from base."""
    at = {a: i for i, (a, *_) in enumerate(insns)}
    seen, work, worst = {}, [(0, -1)], -1  # state: barriers since the oldest read, -1: none
    while work:
        i, state = work.pop()
        if i >= len(insns) or seen.get(i, -2) >= state:
            continue
        seen[i] = state
        _, op, args, line = insns[i]
        if op.startswith("ds_read"):
            state = max(state, 0)
        elif op == "s_waitcnt" and "lgkmcnt(0)" in args:
            state = -1
        elif op == "s_barrier" and state >= 0:
            state = min(state + 1, 3)
            worst = max(worst, state)
        if op == "s_endpgm":
            continue
        if op.startswith("s_cbranch") or op == "s_branch":
            m = TARGET.search(line)
            assert m, line
            work.append((at[base + int(m.group(1) or "0", 16)], state))
        if op != "s_branch":
            work.append((i + 1, state))
    return worst


def kernels(text):
    name, base, insns = None, 0, []
    for line in text.splitlines():
        m = LABEL.match(line)
        if m:
            if name:
                yield name, base, insns
            name, base, insns = m.group(2), int(m.group(1), 16), []
            continue
        m = INSN.match(line)
        if m and name:
            insns.append((int(m.group(3), 16), m.group(1), m.group(2), line))
    if name:
        yield name, base, insns


def test_path_walk_sees_a_read_over_two_barriers():
    """The walk itself, on a prologue with and without its wait (one path skips a barrier)."""
    def prog(*ops):
        return [(4 * i, op.split()[0], op, op) for i, op in enumerate(ops)]
    body = ("s_barrier", "ds_read_b128 v0, v1", "{}", "s_cbranch_scc1 <k+0x14>", "s_barrier",
            "s_barrier", "s_waitcnt lgkmcnt(0)", "s_endpgm")
    missing = prog(*(op.format("s_nop 0") for op in body))
    waited = prog(*(op.format("s_waitcnt lgkmcnt(0)") for op in body))
    assert barriers_over_reads(missing, 0) == 2
    assert barriers_over_reads(waited, 0) == -1


@pytest.mark.skipif(OBJDUMP is None, reason="needs ROCm's llvm-objdump")
def test_no_lds_read_of_the_alternating_tiles_is_in_flight_over_two_barriers(tmp_path):
    lib = shutil.copy(LIB, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", lib], cwd=tmp_path, check=True, capture_output=True)
    found = {}
    for part in sorted(tmp_path.glob("lib.so.*gfx950")):
        text = subprocess.run([OBJDUMP, "-d", str(part)], check=True, capture_output=True,
                              text=True).stdout
        for name, base, insns in kernels(text):
            if "PpTile" in name or "PpBwdTile" in name:
                found[name] = barriers_over_reads(insns, base)
    assert len(found) >= 5, found  # gate+up (whole and mixed), Q/K/V, both [K, N] forms, SwiGLU bwd
    assert all(v == 1 for v in found.values()), found
