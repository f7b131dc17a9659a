"""Wait states around the matrix instructions that csrc/attn_common.h writes as inline assembly, for which the compiler inserts
none: in the built library no vector instruction may write an operand of a 16x16x32 MFMA in the two wait states before it, nor read
or write its result in the eight after it.  (A C compiler's own matrix instructions satisfy the same rules.)  CPU only: reads
the disassembly of the library that build() made."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2510_12872_amd.build import LIB

OBJDUMP = shutil.which("llvm-objdump") or "/opt/rocm/llvm/bin/llvm-objdump"
MFMA = "v_mfma_f32_16x16x32_bf16"
BEFORE, AFTER = 2, 8


def _kernels(tmp_path):
    lib = shutil.copy(LIB, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", str(lib)], check=True, capture_output=True, cwd=tmp_path)
    for name in sorted(os.listdir(tmp_path)):
        if "amdgcn" not in name:
            continue
        text = subprocess.run([OBJDUMP, "-d", str(tmp_path / name)], check=True, capture_output=True, text=True).stdout
        for part in re.split(r"\n(?=[0-9a-f]{16} <)", text):
            if MFMA in part:
                yield part


def _regs(operand):
    m = re.fullmatch(r"-?\|?([va])(?:(\d+)|\[(\d+):(\d+)\])\|?", operand)
    if not m:
        return set()
    lo = int(m[2] or m[3])
    return {m[1] + str(i) for i in range(lo, int(m[2] or m[4]) + 1)}


def parse(part):
    """[(opcode, written registers, read registers, wait states, branch target or None)]"""
    base = int(part[:16], 16)
    code, index = [], {}
    for line in part.split("\n"):
        m = re.match(r"\s+(\S+)\s*(.*?)\s*//\s*([0-9A-F]+):\s*[0-9A-F ]+(?:<[^+>]*(?:\+0x([0-9a-f]+))?>)?", line)
        if not m:
            continue
        op, ops = m[1], [o.strip().split(" ")[0] for o in m[2].split(",")]
        writes, reads = set(), set()
        if op.startswith("v_"):
            both = "swap" in op
            writes = _regs(ops[0]) | (_regs(ops[1]) if both else set())
            reads = set().union(*[_regs(o) for o in ops[0 if both or "fmac" in op or "pk_fmac" in op else 1:]])
        else:
            reads = set().union(*[_regs(o) for o in ops])   # memory instructions: addresses and data
            if re.match(r"(ds_read|global_load|scratch_load|buffer_load)", op):
                writes = _regs(ops[0])
        index[int(m[3], 16)] = len(code)
        target = base + int(m[4], 16) if m[4] and "branch" in op else (base if "branch" in op else None)
        code.append((op, writes, reads, int(ops[0]) + 1 if op == "s_nop" else 1, target))
    return [(o, w, r, n, index.get(t)) for o, w, r, n, t in code]


def ahead(code, i, states):
    """Instructions that can issue within `states` wait states after instruction i."""
    todo, seen = [(i, 0)], {}
    while todo:
        j, dist = todo.pop()
        op, _, _, _, target = code[j]
        nxt = ([] if op in ("s_branch", "s_endpgm") else [j + 1]) + ([target] if target is not None else [])
        for k in nxt:
            if k < len(code) and dist < states and dist < seen.get(k, 99):
                seen[k] = dist
                todo.append((k, dist + code[k][3]))
    return seen


def violations(code):
    bad = []
    for i, (op, writes, _, _, _) in enumerate(code):
        if op == MFMA:
            for k in ahead(code, i, AFTER):
                if not code[k][0].startswith("v_mfma") and writes & (code[k][1] | code[k][2]):
                    bad.append((i, k))
        elif op.startswith("v_") and not op.startswith("v_mfma"):
            for k in ahead(code, i, BEFORE):
                if code[k][0] == MFMA and writes & code[k][2]:
                    bad.append((i, k))
    return bad


def test_wait_states(tmp_path):
    if not os.path.exists(LIB):
        pytest.skip("needs the built library")
    assert os.path.exists(OBJDUMP), "no llvm-objdump: nothing else guards the wait states of a new build"
    n = 0
    for part in _kernels(tmp_path):
        code = parse(part)
        n += sum(c[0] == MFMA for c in code)
        bad = violations(code)
        assert not bad, (part[:120], [(code[i], code[k]) for i, k in bad[:4]])
    assert n > 1000   # the kernels were found


@pytest.mark.parametrize("lines,found", [
    (["v_mov_b32 v4, v9", "X v[0:3], v[4:7], v[8:11], v[0:3]"], True),
    (["v_mov_b32 v4, v9", "s_nop 1", "X v[0:3], v[4:7], v[8:11], v[0:3]"], False),
    (["v_mov_b32 v1, v9", "s_nop 0", "X v[0:3], v[4:7], v[8:11], v[0:3]"], True),
    (["X v[0:3], v[4:7], v[8:11], v[0:3]", "s_nop 6", "v_mov_b32 v9, v3"], True),
    (["X v[0:3], v[4:7], v[8:11], v[0:3]", "s_nop 7", "v_mov_b32 v9, v3"], False),
    (["X a[0:3], v[4:7], v[8:11], a[0:3]", "v_accvgpr_read_b32 v1, a3"], True),
    (["X v[0:3], v[4:7], v[8:11], v[0:3]", "v_mov_b32 v5, v9"], False),   # operands are read at issue
    (["X v[0:3], v[4:7], v[8:11], v[0:3]", "s_branch 1 <k+0x10>", "s_nop 7", "s_nop 7", "v_add_f32 v9, v0, v9"], True),
])
def test_checker(lines, found):
    part = "%016x <k>:\n" % 0 + "\n".join(
        "\t%s // %012X: BF800000%s" % (re.sub(r" <.*>", "", l).replace("X", MFMA), 4 * i, " <k+0x10>" if "<" in l else "")
        for i, l in enumerate(lines)) + "\n\ts_endpgm // %012X: BF800000" % (4 * len(lines))
    assert bool(violations(parse(part))) == found
