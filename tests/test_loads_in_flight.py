"""Registers of loads in flight in the compiled kernels (CPU only: the device code is compiled to assembly with the
build's own flags and read).

Some kernels issue loads by inline assembly and wait for them later, by count, so that other copies stay in flight.
The compiler takes such a register as written at once: nothing but the build's register allocation keeps it from being
copied, spilled or reused before the wait.  The scan follows every path of every kernel with the vector-memory
operations outstanding on it (in issue order; a wait leaves the last N) and reports each instruction that names a
register whose load has not been waited for."""
import os
import re
import subprocess

import pytest

from paper_2606_00535_amd import build

MEMORY = re.compile(r"(global|buffer|flat|scratch)_(load|store|atomic)")
REGISTER = re.compile(r"\bv\[(\d+):(\d+)\]|\bv(\d+)\b")


def registers(text):
    return {r for m in REGISTER.finditer(text)
            for r in (range(int(m[1]), int(m[2]) + 1) if m[1] else (int(m[3]),))}


def kernels(assembly):
    """{name: [(label or None, instruction, whether by inline assembly), ...]} of every kernel."""
    out = {}
    for m in re.finditer(r"^(\w+):[^\n]*; @\1\n(.*?)^\.Lfunc_end", assembly, re.M | re.S):
        code, inline = [], False
        for line in m[2].split("\n"):
            inline = "#ASMSTART" in line or (inline and "#ASMEND" not in line)
            line = line.split(";")[0].strip()
            if re.match(r"\.LBB\w+:", line):
                code.append((line[:-1], None, False))
            elif line and not line.startswith("."):
                code.append((None, line, inline))
        out[m[1]] = code
    return out


def scan(code, limit=50000):
    """The instructions of one kernel that touch a register that inline assembly is loading, and how many such loads
    there are.  (The compiler waits for its own.)

    A path's state is the set of (operations issued since, registers) of the loads it has not waited for: a wait
    for all but N leaves those with fewer than N issued since (counted up to 64: no wait can leave more)."""
    at = {label: i for i, (label, _, _) in enumerate(code) if label}
    ops = []                         # per line: what it is, the registers it names, those it loads into, its argument
    loads = 0
    for label, text, inline in code:
        if label:
            ops.append(("label", frozenset(), frozenset(), None))
            continue
        op = text.split()[0]
        kind, into, arg = "other", frozenset(), None
        if MEMORY.match(op):
            kind = "memory"
            if inline and "_load" in op and "_lds_" not in op:
                into = frozenset(registers(text.split(None, 1)[1].split(",")[0]))
                loads += 1
        elif op == "s_waitcnt":
            m = re.search(r"vmcnt\((\d+)\)", text)
            kind, arg = ("wait", int(m[1])) if m else ("other", None)
        elif op == "s_endpgm":
            kind = "end"
        elif op == "s_branch" or op.startswith("s_cbranch"):
            kind, arg = ("jump" if op == "s_branch" else "branch"), at[text.split()[1]]
        ops.append((kind, frozenset(registers(text)), into, arg))
    bad, seen, todo = {}, set(), [(0, frozenset())]
    while todo:
        i, flight = todo.pop()
        while i < len(ops):
            kind, named, into, arg = ops[i]
            if kind == "label":
                if (i, flight) in seen:
                    break
                seen.add((i, flight))
                assert len(seen) < limit, "too many paths"
            elif kind == "wait":
                flight = frozenset(f for f in flight if f[0] < arg)
            elif kind == "end":
                break
            elif kind in ("jump", "branch"):
                todo.append((arg, flight))
                if kind == "jump":
                    break
            else:
                if any(named & regs for _, regs in flight):
                    bad[i] = code[i][1]
                if kind == "memory":
                    flight = frozenset((min(n + 1, 64), regs) for n, regs in flight)
                    if into:
                        flight |= {(0, into)}
            i += 1
    return [bad[i] for i in sorted(bad)], loads


def assembly_of(name, tmp):
    out = os.path.join(str(tmp), name + ".s")
    r = subprocess.run([build.HIPCC] + build.CFLAGS + ["--cuda-device-only", "-S", os.path.join(build.CSRC, name + ".hip"),
                                                      "-o", out], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return open(out).read()


def sources_with_assembly_loads():
    found = [os.path.basename(s)[:-4] for s in build.sources()
             if re.search(r'asm[^;]*"(global|buffer|flat)_load_(?!lds)', open(s).read())]
    assert "prefill_stats" in found
    return found


needs_compiler = pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="hipcc is not installed")


@needs_compiler
@pytest.mark.parametrize("name", sources_with_assembly_loads())
def test_no_register_is_touched_while_its_load_is_in_flight(name, tmp_path):
    found, total = kernels(assembly_of(name, tmp_path)), 0
    for kernel, code in found.items():
        bad, loads = scan(code)
        assert not bad, "%s: %s" % (kernel, bad[:5])
        total += loads
    assert total


SAMPLE = """
kernel: ; @kernel
	global_load_lds_dwordx4 v[0:1], off
	;;#ASMSTART
	global_load_dwordx4 v[4:7], v[0:1], off
	;;#ASMEND
	global_load_lds_dwordx4 v[2:3], off
.LBB0_1:
	s_cbranch_scc1 .LBB0_3
	s_waitcnt vmcnt(1)
	ds_write_b128 v8, v[4:7]
.LBB0_3:
	s_endpgm
.Lfunc_end0:
"""


@pytest.mark.parametrize("before,after,bad", [
    ("", "", 0),
    ("vmcnt(1)", "vmcnt(2)", 1),                                     # a wait that leaves the load in flight
    ("\ts_waitcnt vmcnt(1)\n", "", 1),                               # none
    (".LBB0_1:\n", "\tv_mov_b32_e32 v9, v6\n.LBB0_1:\n", 1),         # a copy of a register in flight
    (".LBB0_1:\n", "\tv_mov_b32_e32 v5, 0\n.LBB0_1:\n", 1),          # its reuse
    (".LBB0_3:\n", ".LBB0_3:\n\tv_add_u32_e32 v9, v4, v4\n", 1),     # a use that one of two paths waits for
    ("v[2:3], off", "v[6:7], off", 1),                               # as another copy's address
    ("\t;;#ASMSTART\n", "", 0),                                      # the compiler's own load
])
def test_the_scan_sees(before, after, bad):
    assert len(scan(kernels(SAMPLE.replace(before, after, 1) if before else SAMPLE)["kernel"])[0]) == bad
