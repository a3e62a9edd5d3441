"""Wait states of the kernels that load straight into LDS, in the assembly
hipcc makes of them here.

A vector-memory instruction must not read an SGPR within five wait states of
the vector instruction that wrote it (v_readlane_b32, v_readfirstlane_b32,
compares into SGPRs).  The compiler keeps that distance for its own memory
instructions but does not look into inline assembly, so the assembly of
sw_device.h has to bring its own wait states.  Nor can it say that it writes
M0 (a reserved register): the compiler's own instructions must not use it.
"""
import concurrent.futures
import os
import re
import subprocess

import pytest

from paper_2609_34117_amd import build

WAIT_STATES = 5
_SGPR = re.compile(r"\bs(\d+)\b|\bs\[(\d+):(\d+)\]")
_VMEM = re.compile(r"(buffer|global|flat|scratch|tbuffer)_")


def _sgprs(text):
    regs = set()
    for one, lo, hi in _SGPR.findall(text):
        regs.update([int(one)] if one else range(int(lo), int(hi) + 1))
    return regs


class Inst:
    def __init__(self, text):
        self.op, _, args = text.partition(" ")
        self.text = text
        ops = [o.strip() for o in args.split(",")]
        vector = self.op.startswith("v_")
        n_dst = 2 if vector and ("_co_" in self.op or "div_scale" in self.op or "_mad_u64" in self.op
                                 or "_mad_i64" in self.op) else 1
        self.writes = _sgprs(" ".join(ops[:n_dst])) if vector or self.op.startswith("s_") else set()
        self.vector_writes = self.writes if vector else set()
        self.vmem_reads = _sgprs(args) if _VMEM.match(self.op) else set()
        self.states = int(ops[0]) + 1 if self.op == "s_nop" else 1
        self.target = ops[0] if self.op.startswith(("s_branch", "s_cbranch")) else None
        self.ends = self.op in ("s_endpgm", "s_branch")


def parse(asm):
    """Instructions in order, and the index each label stands for."""
    insts, labels = [], {}
    for line in asm.splitlines():
        line = line.split(";")[0].strip()
        if re.fullmatch(r"[\w.$]+:", line):
            labels[line[:-1]] = len(insts)
        elif line and line[0] not in ".#" and re.match(r"[a-z]\w*(\s|$)", line):
            insts.append(Inst(re.sub(r"\s+", " ", line)))
    return insts, labels


def too_close(asm):
    """(writer, reader, wait states between) of every vector-memory
    instruction that reads an SGPR too soon after a vector write of it, along
    fall-through and branches."""
    insts, labels = parse(asm)
    found = {}
    for i, w in enumerate(insts):
        if not w.vector_writes:
            continue
        walk = [(i + 1, 0, frozenset(w.vector_writes))]
        while walk:
            j, gone, regs = walk.pop()
            while j < len(insts) and gone < WAIT_STATES and regs:
                n = insts[j]
                if n.vmem_reads & regs:
                    found[j] = (w.text, n.text, gone)
                gone += n.states
                regs = regs - n.writes
                if n.target in labels:
                    walk.append((labels[n.target], gone, regs))
                if n.ends:
                    break
                j += 1
    return list(found.values())


def compilers_own_m0(asm):
    """In functions with LDS loads in inline assembly, the instructions outside
    it that name M0."""
    found = []
    for function in asm.split("; -- Begin function"):
        inline, own, loads = False, [], False
        for line in function.splitlines():
            text = line.strip()
            if text == ";;#ASMSTART":
                inline = True
            elif text == ";;#ASMEND":
                inline = False
            elif inline:
                loads = loads or text.endswith(" lds")
            elif re.search(r"\bm0\b", text.split(";")[0]):
                own.append(text)
        if loads:
            found += own
    return found


def _assembly(src):
    r = subprocess.run([build.HIPCC, *build.HIP_FLAGS, "--cuda-device-only", "-S", src, "-o", "-"],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    return r.stdout


def test_scanner_sees_the_distance():
    lds = "buffer_load_dword v0, s[40:43], 0 offen lds\n"
    short = "v_readlane_b32 s43, v1, 2\ns_mov_b32 m0, s5\ns_nop 0\n" + lds
    assert [d for *_, d in too_close(short)] == [2]
    assert not too_close(short.replace("s_nop 0", "s_nop 3"))
    assert not too_close(short.replace("s_nop 0", "s_mov_b32 s43, 0"))  # another writer since
    over_branch = "L:\ns_nop 2\n" + lds + "v_readfirstlane_b32 s40, v1\ns_branch L\n"
    assert [d for *_, d in too_close(over_branch)] == [4]
    load = ";;#ASMSTART\ns_mov_b32 m0, s5\n" + lds + ";;#ASMEND\ns_nop 0 ; m0\n"
    own = "\ts_mov_b32 m0, s5\n"
    assert not compilers_own_m0(load + "; -- Begin function f\n" + own)
    assert len(compilers_own_m0(own + "; -- Begin function f\n" + load + own)) == 1


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="needs hipcc")
def test_lds_loads_keep_their_wait_states_and_m0():
    srcs = [s for s in build.sources() if re.search(r"\bload_lds(4|16)\b", open(s).read())]
    assert len(srcs) >= 2
    with concurrent.futures.ThreadPoolExecutor(max_workers=4) as ex:
        for src, asm in zip(srcs, ex.map(_assembly, srcs)):
            assert re.search(r"buffer_load_dwordx4 .* lds\b", asm), src
            bad = too_close(asm)
            assert not bad, (os.path.basename(src), len(bad), bad[:4])
            own = compilers_own_m0(asm)
            assert not own, (os.path.basename(src), len(own), own[:4])
