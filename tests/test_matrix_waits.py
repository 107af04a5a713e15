"""Waits after matrix instructions in the built library (CPU).

The hardware does not hold back an instruction that reads the registers of a
matrix instruction still in flight: the compiler has to place wait states.
hipcc 7.2 has left them out where the first reader stands behind a branch, and
the results were wrong on the GPU only.  The test disassembles the device code
that was built here and follows every path of every kernel from each matrix
instruction, for as many wait states as the compiler itself places in straight
code for gfx950: FP64 16x16x4 19 before a vector or matrix operand and 18 before
a memory operand, FP32 16x16x4 10 before any.
"""
import os
import re
import shutil
import subprocess

import pytest

from paper_1807_00370_amd import _lib, build

LLVM = "/opt/rocm/llvm/bin"
TARGET = "hipv4-amdgcn-amd-amdhsa--gfx950"
MEMORY = ("global_", "flat_", "scratch_", "buffer_", "ds_")
NO_RESULT = ("global_store", "flat_store", "scratch_store", "buffer_store", "ds_write", "global_atomic")


def _regs(text):
    """Vector registers named in operand text (accumulation registers from 1000)."""
    out = set()
    for kind, a, b in re.findall(r"\b([va])\[(\d+):(\d+)\]", text):
        out |= {int(q) + (1000 if kind == "a" else 0) for q in range(int(a), int(b) + 1)}
    for kind, a in re.findall(r"\b([va])(\d+)\b", text):
        out.add(int(a) + (1000 if kind == "a" else 0))
    return out


def _functions(dis):
    """name -> list of (opcode, operands, written, read, branch target index)."""
    for part in re.split(r"^[0-9a-f]+ <", dis, flags=re.M)[1:]:
        name, body = part.split(">:", 1)
        base, ins, at, jumps = None, [], {}, {}
        for line in body.splitlines():
            m = re.match(r"\s+(\S+)\s*(.*?)\s*// ([0-9A-F]+):", line)
            if not m:
                continue
            op, args, addr = m.group(1), m.group(2), int(m.group(3), 16)
            base = addr if base is None else base
            at[addr - base] = len(ins)
            if op.startswith(("s_branch", "s_cbranch")):
                jumps[len(ins)] = int(re.search(r"\+0x([0-9a-f]+)>\s*$", line).group(1), 16) \
                    if "+0x" in line.rsplit("<", 1)[-1] else 0
            ops = [q.strip() for q in re.split(r",(?![^\[]*\])", args)]
            none = op.startswith(NO_RESULT) or op.startswith(("s_", "v_cmp", "v_read"))
            written = set() if none or not args else _regs(ops[0])
            read = _regs(", ".join(ops if none else ops[1:]))
            ins.append([op, args, written, read, None])
        for i, target in jumps.items():
            ins[i][4] = at[target]  # a jump out of the kernel would raise here
        yield name, ins


def early_reads(dis):
    """[(kernel, matrix instruction, reader)] that come too early on some path."""
    bad = []
    for name, ins in _functions(dis):
        for i, (op, args, written, _, _) in enumerate(ins):
            if not op.startswith("v_mfma"):
                continue
            vec, mem = (19, 18) if "f64" in op else (10, 10)
            todo, seen = [(i + 1, 0, frozenset(written))], set()
            while todo:
                j, w, live = todo.pop()
                while j < len(ins) and w < vec and live and (j, w, live) not in seen:
                    seen.add((j, w, live))
                    o, a, wr, rd, target = ins[j]
                    if o.startswith("v_mfma"):
                        # an accumulator is taken over in the matrix pipeline
                        ops = [q.strip() for q in re.split(r",(?![^\[]*\])", a)]
                        rd = _regs(ops[1]) | _regs(ops[2])
                    if rd & live and w < (mem if o.startswith(MEMORY) else vec):
                        bad.append((name, op + " " + args, o + " " + a))
                        live = live - rd
                    live = live - wr
                    if o == "s_endpgm":
                        break
                    w += int(a, 0) + 1 if o == "s_nop" else 1
                    # a taken branch refills the instruction buffer: two states
                    # at the least
                    if o == "s_branch":
                        j, w = target, w + 1
                        continue
                    if target is not None:
                        todo.append((target, w + 1, live))
                    j += 1
    return bad


def _disassemble(lib, tmp):
    fat, obj = os.path.join(tmp, "fat"), os.path.join(tmp, "obj")
    run = lambda *a: subprocess.run(a, check=True, capture_output=True, text=True).stdout
    run(LLVM + "/llvm-objcopy", "-O", "binary", "--only-section=.hip_fatbin", lib, fat)
    run(LLVM + "/clang-offload-bundler", "--unbundle", "--type=o", "--targets=" + TARGET,
        "--input=" + fat, "--output=" + obj)
    return run(LLVM + "/llvm-objdump", "-d", "--no-show-raw-insn", obj)


def test_scan_finds_a_missing_wait():
    """The scan itself: a reader behind a branch, with and without waits."""
    text = """
0000000000001000 <k>:
\tv_mfma_f64_16x16x4_f64 v[0:7], v[8:9], v[10:11], 0 // 000000001000: 00
\ts_cbranch_scc1 2 // 000000001008: 00 <k+0x14>
\ts_nop %s // 00000000100C: 00
\ts_endpgm // 000000001010: 00
\tv_add_f64 v[12:13], v[2:3], 1.0 // 000000001014: 00
\ts_endpgm // 00000000101C: 00
"""
    assert [b[2] for b in early_reads(text % 15)] == ["v_add_f64 v[12:13], v[2:3], 1.0"]
    waits = text.replace("\ts_cbranch", "\ts_nop 15 // 000000001004: 00\n\ts_nop 1 // 000000001006: 00\n\ts_cbranch")
    assert early_reads(waits % 0) == []


def test_no_matrix_result_is_read_early(tmp_path):
    if not os.path.exists(_lib.LIB_PATH):
        build.build_library()
    if not shutil.which(LLVM + "/llvm-objdump"):
        pytest.skip("no disassembler")
    dis = _disassemble(_lib.LIB_PATH, str(tmp_path))
    assert dis.count("v_mfma") > 1000
    bad = early_reads(dis)
    assert not bad, "%d early reads, first: %s" % (len(bad), bad[:3])
