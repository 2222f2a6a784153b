"""The product kernels (csrc/kd_products.hip) run on the strip loop with operand fragments that inline assembly reads from
LDS in two halves, which neither the compiler's hazard nor its wait handling sees.  This test reads the gfx950 code of the
built library and checks, along every path, the MFMA hazards of test_strip_hazards.py and that nothing touches a register
that an LDS read still has to fill."""
import re
import subprocess

from paper_2603_01875_amd import kdloss as K
from tests.test_strip_hazards import LLVM, MFMA, _code_objects, _regs, hazards, parse

KERNELS = r"grad_[wh]_kernel"


def early_uses(code):
    """(address, what) of every instruction that touches a register whose LDS read may be in flight.  LDS reads land in
    order; s_waitcnt lgkmcnt(n) leaves at most the n youngest."""
    at = {c.addr: i for i, c in enumerate(code)}
    found, todo, seen = set(), [(0, ())], set()
    while todo:
        i, flying = todo.pop()
        if (i, flying) in seen:
            continue
        seen.add((i, flying))
        flying = list(flying)
        while True:
            c = code[i]
            if c.op.startswith("ds_read"):
                new = _regs(c.operands[0])
                if any(r in f for f in flying for r in c.touched - new):
                    found.add((c.addr, "address in flight"))
                flying = (flying + [frozenset(new)])[-40:]
            elif any(r in f for f in flying for r in c.touched):
                found.add((c.addr, c.op))
            elif c.op == "s_waitcnt":
                m = re.search(r"lgkmcnt\((\d+)\)", " ".join(c.operands))
                if m:
                    flying = flying[max(0, len(flying) - int(m[1])):]
            if c.op == "s_endpgm":
                break
            if c.target in at and c.op.startswith(("s_cbranch", "s_branch")):
                todo.append((at[c.target], tuple(flying)))
                if c.op.startswith("s_branch"):
                    break
                todo.append((i + 1, tuple(flying)))
                break
            i += 1
    return sorted(found)


def test_no_hazard_in_the_product_kernels(tmp_path):
    K.lib()
    kernels = {}
    for obj in _code_objects(K._LIB_PATH, str(tmp_path)):
        text = subprocess.run([f"{LLVM}/llvm-objdump", "-d", "--no-show-raw-insn", obj], check=True, capture_output=True,
                              text=True).stdout
        for m in re.finditer(r"^([0-9a-f]+) <(\S*%s\S*)>:\n((?:\t.*\n)+)" % KERNELS, text, re.M):
            kernels[m[2]] = parse(m[3].splitlines(), int(m[1], 16))
    assert len(kernels) == 24 + 8             # grad_W_s: 3 tiles x order x type x add; grad_h_s: 4 tiles x order
    for name, code in kernels.items():
        assert sum("ds_read_b64" in c.op for c in code) >= 2 * 2 * 4, name
        assert hazards(code) == [], name
        assert early_uses(code) == [], name


def test_the_check_sees_planted_early_uses():
    read = "ds_read_b64_tr_b16 v[0:1], v9"
    for text, n in [([read, MFMA], 1), ([read, "s_waitcnt lgkmcnt(0)", MFMA], 0), ([read, "v_mov_b32_e32 v20, v1"], 1),
                    ([read, "ds_read_b64 v[20:21], v9", "s_waitcnt lgkmcnt(1)", MFMA], 0),
                    ([read, "ds_read_b64 v[2:3], v9", "s_waitcnt lgkmcnt(1)", MFMA], 1),
                    # the read in flight is only met through the jump back
                    ([MFMA, read, "s_cbranch_scc0 9 <+0>"], 1)]:
        lines = []
        for i, t in enumerate(text + ["s_endpgm"]):
            t, _, target = t.partition(" <+")
            lines.append(f"\t{t}   // {4 * i:012X}: 00000000" + (f" <k+0x{target[:-1]}>" if target else ""))
        assert len(early_uses(parse(lines, 0))) == n, text
