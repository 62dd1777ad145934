"""Wait states between a matrix instruction and the first vector or memory
instruction that touches its result, over every path of the built kernels.

The hardware does not hold such a reader back: on gfx950 the 16x16 products
used here (four passes) need 8 wait states, an instruction or an s_nop count
each, and the compiler counts them.  Sums of such results that it moved past a
branch have come out with fewer on the taken path, so the built code is read
back: straight-line code shows 8 everywhere.  Skipped where the library is not
built.
"""

import os
import re
import shutil
import subprocess

import pytest

from paper_2609_33410_amd import build_lib

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
NEED = 8
FOUR_PASS = {"v_mfma_f32_16x16x16_bf16", "v_mfma_f32_16x16x32_bf16", "v_mfma_f32_16x16x32_f16",
             "v_mfma_i32_16x16x64_i8"}
MEMORY = ("ds_", "buffer_", "global_", "flat_", "scratch_")


def _regs(text):
    """Vector registers named in some operands (accumulation registers from 512)."""
    out = set()
    for bank, lo, hi, one in re.findall(r"(?<!\w)([va])(?:\[(\d+):(\d+)\]|(\d+)\b)", text):
        base = 512 if bank == "a" else 0
        a, b = (int(one), int(one)) if one else (int(lo), int(hi))
        out.update(range(base + a, base + b + 1))
    return out


def early_reads(code):
    """(product, reader, wait states) of every read or overwrite of a matrix
    result less than NEED wait states after it.  code: (mnemonic, operands,
    branch target index or None) in order."""
    found = []
    for i, (op, args, _) in enumerate(code):
        if not op.startswith("v_mfma"):
            continue
        assert op in FOUR_PASS, f"{op}: its passes are not known here"
        todo, seen = [(i + 1, 0, frozenset(_regs(args.split(",")[0])))], set()
        while todo:
            at, waits, live = todo.pop()
            if waits >= NEED or at >= len(code) or not live or (at, waits) in seen:
                continue
            seen.add((at, waits))
            rop, rargs, target = code[at]
            if rop == "s_endpgm":
                continue
            if rop.startswith("v_mfma"):  # C may be taken early; A and B may not
                parts = rargs.split(", ")
                hit = (_regs(parts[1]) | _regs(parts[2])) & live
                live = live - _regs(parts[0])
            else:
                hit = _regs(rargs) & live if rop.startswith(("v_",) + MEMORY) else set()
            if hit:
                found.append((op, f"{rop} {rargs}", waits))
                live = live - hit
            step = int(rargs, 0) + 1 if rop == "s_nop" else 1
            if target is not None:
                todo.append((target, waits + step, live))
            if rop != "s_branch":
                todo.append((at + 1, waits + step, live))
    return found


def _functions(asm):
    """name -> code of a disassembly (llvm-objdump -d)."""
    out = {}
    for name, body in re.findall(r"^[0-9a-f]+ <([^>]+)>:\n(.*?)(?=^[0-9a-f]+ <|\Z)", asm,
                                 re.S | re.M):
        rows = []
        for line in body.splitlines():
            m = re.match(r"\s+([a-z]\w+)\s*(.*?)\s*// ([0-9A-F]+):[^<]*(?:<[^>+]+(?:\+0x([0-9a-f]+))?>)?",
                         line)
            if m:
                rows.append((m.group(1), m.group(2), int(m.group(3), 16), m.group(4)))
        index = {r[2]: k for k, r in enumerate(rows)}
        base = rows[0][2] if rows else 0
        out[name] = [(op, args, index.get(base + int(off or "0", 16))
                      if op.startswith(("s_branch", "s_cbranch")) else None)
                     for op, args, _, off in rows]
    return out


def test_finds_a_read_past_a_taken_branch():
    """Nine instructions on the way through, none past the taken branch."""
    mfma = ("v_mfma_i32_16x16x64_i8", "v[0:3], v[8:11], v[12:15], 0", None)
    fill = ("v_mov_b32_e32", "v20, 0", None)
    read = ("v_add_u32_e32", "v5, v6, v3", None)
    end = ("s_endpgm", "", None)
    code = [mfma, ("s_cbranch_vccnz", "9", 11)] + [fill] * 9 + [read, end]
    assert [w for _, _, w in early_reads(code)] == [1]
    code[1:2] = [("s_nop", "6", None), ("s_cbranch_vccnz", "9", 12)]
    assert early_reads(code) == []


def test_built_kernels_wait_for_their_matrix_results(tmp_path):
    if not os.path.exists(build_lib.LIB):
        pytest.skip("the library is not built")
    if not os.path.exists(OBJDUMP):
        pytest.skip("no disassembler")
    lib = str(tmp_path / "libfold.so")
    shutil.copy(build_lib.LIB, lib)
    subprocess.run([OBJDUMP, "--offloading", lib], check=True, stdout=subprocess.DEVNULL)
    objects = sorted(tmp_path.glob("*gfx950*"))
    assert len(objects) == sum(s.endswith(".hip") for s in build_lib.SOURCES)
    products = 0
    for obj in objects:
        asm = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(obj)], check=True,
                             capture_output=True, text=True).stdout
        for name, code in _functions(asm).items():
            products += sum(op.startswith("v_mfma") for op, _, _ in code)
            assert all(t is not None for op, _, t in code if op.startswith("s_cbranch"))
            assert early_reads(code) == [], name
    assert products > 1000  # the disassembly was read
