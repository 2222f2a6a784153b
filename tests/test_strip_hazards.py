"""The strip loop's MFMAs are inline assembly, so the compiler puts no wait states between them and what touches their
registers (csrc/kd_strip.hpp).  This test reads the gfx950 code of the built library and checks, along every path through
every strip kernel, that
  - no vector instruction writes an operand of an MFMA within the two slots before it, and
  - nothing but an MFMA accumulating into the same registers touches an MFMA's result within the sixteen slots after it
(a slot is an instruction; s_nop n counts as n + 1).  The needs of these 16x16x32 MFMAs are smaller than both numbers."""
import collections
import os
import re
import struct
import subprocess

import pytest

from paper_2603_01875_amd import kdloss as K

LLVM = "/opt/rocm/llvm/bin"
BEFORE, AFTER = 2, 16
REG = re.compile(r"\b([va])(?:(\d+)\b|\[(\d+):(\d+)\])")
LINE = re.compile(r"^\t(\S+)(?: ([^/]*))?\s*// ([0-9A-F]+):[0-9A-F ]*(?:<\S+\+0x([0-9a-f]+)>)?")
Inst = collections.namedtuple("Inst", "op operands touched addr target")


def _regs(text):
    out = set()
    for m in REG.finditer(text):
        lo, hi = (int(m[2]), int(m[2])) if m[2] else (int(m[3]), int(m[4]))
        out.update((m[1], i) for i in range(lo, hi + 1))
    return out


def parse(lines, base):
    out = []
    for line in lines:
        if line.strip() == "...":              # zeros between two kernels
            continue
        m = LINE.match(line)
        assert m, line
        ops = [o.strip() for o in (m[2] or "").split(",")]
        out.append(Inst(m[1], ops, frozenset(_regs(m[2] or "")), int(m[3], 16), base + int(m[4], 16) if m[4] else None))
    return out


def hazards(code):
    """(address, what) of every violation in one kernel; `code` is a list of Inst in address order."""
    at = {c.addr: i for i, c in enumerate(code)}
    jumps = [i for i, c in enumerate(code) if c.op.startswith(("s_cbranch", "s_branch"))]
    assert all(code[i].target in at for i in jumps)
    leaders = sorted({0} | {at[code[i].target] for i in jumps} | {i + 1 for i in jumps if i + 1 < len(code)})
    ends = leaders[1:] + [len(code)]
    entry = {b: ({}, {}) for b in leaders}       # register -> slots still to pass: MFMA results, vector results
    found, todo, seen = set(), [0], set()
    while todo:
        b = todo.pop()
        seen.add(b)
        end = ends[leaders.index(b)]
        results, writes = (dict(d) for d in entry[b])
        slot = 0
        for c in code[b:end]:
            mfma = c.op.startswith("v_mfma")
            if mfma:
                dst, acc = _regs(c.operands[0]), _regs(c.operands[3])
                src = _regs(c.operands[1]) | _regs(c.operands[2])
                if any(writes.get(r, 0) > slot for r in c.touched):
                    found.add((c.addr, "operand written just before " + c.op))
                if any(results.get(r, 0) > slot for r in src) or (acc != dst and any(results.get(r, 0) > slot for r in acc)):
                    found.add((c.addr, "result read by another MFMA too early"))
            elif c.touched and any(results.get(r, 0) > slot for r in c.touched):
                found.add((c.addr, "result touched too early by " + c.op))
            slot += int(c.operands[0], 0) + 1 if c.op == "s_nop" else 1
            if mfma:
                results.update((r, slot + AFTER) for r in dst)
            elif c.op.startswith("v_"):
                both = 2 if "swap" in c.op else 1
                writes.update((r, slot + BEFORE) for o in c.operands[:both] for r in _regs(o))
        last = code[end - 1]
        nxt = [at[last.target]] if last.target is not None and last.op.startswith(("s_cbranch", "s_branch")) else []
        if not last.op.startswith(("s_branch", "s_endpgm")) and end < len(code):
            nxt.append(end)
        for n in nxt:
            grown = n not in seen
            for have, out in zip(entry[n], (results, writes)):
                for r, s in out.items():
                    if s - slot > have.get(r, 0):
                        have[r], grown = s - slot, True
            if grown and n not in todo:
                todo.append(n)
    return sorted(found)


def _code_objects(path, tmp):
    fat = os.path.join(tmp, "fat.bin")
    subprocess.run([f"{LLVM}/llvm-objcopy", "--dump-section", f".hip_fatbin={fat}", path, os.devnull], check=True)
    data, magic = open(fat, "rb").read(), b"__CLANG_OFFLOAD_BUNDLE__"
    pos = data.find(magic)
    while pos >= 0:
        n, p = struct.unpack_from("<Q", data, pos + 24)[0], pos + 32
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + length]:
                name = os.path.join(tmp, f"{pos}.o")
                open(name, "wb").write(data[pos + off:pos + off + size])
                yield name
            p += 24 + length
        pos = data.find(magic, pos + 24)


def test_no_hazard_in_the_strip_kernels(tmp_path):
    K.lib()
    kernels = {}
    for obj in _code_objects(K._LIB_PATH, str(tmp_path)):
        text = subprocess.run([f"{LLVM}/llvm-objdump", "-d", "--no-show-raw-insn", obj], check=True, capture_output=True,
                              text=True).stdout
        for m in re.finditer(r"^([0-9a-f]+) <(\S*strip_kernel\S*)>:\n((?:\t.*\n)+)", text, re.M):
            kernels[m[2]] = parse(m[3].splitlines(), int(m[1], 16))
    assert len(kernels) == 17                 # statistics x 4, rows x 5, gradient x 7, the AKL search
    for name, code in kernels.items():
        assert sum(c.op.startswith("v_mfma") for c in code) >= 4 * 48, name
        assert hazards(code) == [], name


MFMA = "v_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[4:7], a[0:3]"


@pytest.mark.parametrize("text, n", [
    ([MFMA, MFMA], 0), (["v_mov_b32_e32 v4, v9", MFMA], 1), (["v_mov_b32_e32 v4, v9", "s_nop 1", MFMA], 0),
    (["v_permlane32_swap_b32_e32 v9, v7", "s_nop 0", MFMA], 1), ([MFMA, "s_nop 14", "v_accvgpr_read_b32 v9, a2"], 1),
    ([MFMA, "s_nop 15", "v_accvgpr_read_b32 v9, a2"], 0), ([MFMA, "ds_write_b128 v9, a[0:3]"], 1),
    ([MFMA, MFMA.replace("v[0:3]", "a[0:3]")], 1),
    # the second is only reached through the jump back over it
    (["s_branch 2 <+8>", "v_accvgpr_read_b32 v9, a2", MFMA, "s_cbranch_scc0 9 <+4>", "s_endpgm"], 1)])
def test_the_check_sees_planted_hazards(text, n):
    lines = []
    for i, t in enumerate(text):
        t, _, target = t.partition(" <+")
        lines.append(f"\t{t}   // {4 * i:012X}: 00000000" + (f" <k+0x{target[:-1]}>" if target else ""))
    assert len(hazards(parse(lines, 0))) == n
