"""The product kernels (csrc/kd_products.hip) run on the strip loop with operand fragments that inline assembly reads from
LDS in two halves, which neither the compiler's hazard nor its wait handling sees.  This test reads the gfx950 code of the
built library and checks, along every path, the MFMA hazards of test_strip_hazards.py and that nothing touches a register
that an LDS read still has to fill.  grad_w_few_kernel, whose MFMAs are the compiler's, fills its LDS stages by loads that it waits for
by count: no wait may leave a load of the stage that is read next in flight."""
import re
import subprocess

from paper_2603_01875_amd import kdloss as K
from tests.test_strip_hazards import LLVM, MFMA, _code_objects, _regs, hazards, parse

KERNELS = r"grad_(?:[wh]|w_few)_kernel"
PANELS, AHEAD = 4, 3                          # GradWFew: loads a stage and wave, stages in flight


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


def late_waits(code):
    """(barriers seen, addresses of those that stage loads may be late for).  At a barrier the stage of AHEAD - 1 steps may still be on
    its way; the one before it must have landed.  Vector memory operations land in order; s_waitcnt vmcnt(n) leaves at most the
    n youngest in flight.  A wait that counts results, too, stands where AHEAD steps have been made: no path takes it before."""
    at = {c.addr: i for i, c in enumerate(code)}
    barriers, found, todo, seen = set(), set(), [(0, (), 0, 0)], set()
    need = PANELS * (AHEAD - 1) + 1           # the last load of the stage that is read next, counted from the youngest
    while todo:
        state = todo.pop()
        if state in seen:
            continue
        seen.add(state)
        i, since, left, steps = state         # since: operations issued after each of the last stage loads; left: in flight at most
        while True:
            c = code[i]
            if c.op.startswith(("buffer_", "global_", "flat_", "scratch_")):
                since, left = tuple(min(n + 1, 99) for n in since), min(left + 1, 99)
                if any(re.search(r"\blds\b", o) for o in c.operands):
                    since = (since + (0,))[-need:]
            elif c.op == "s_waitcnt":
                m = re.search(r"vmcnt\((\d+)\)", " ".join(c.operands))
                left = min(left, int(m[1])) if m else left
                if m and code[i + 1].op == "s_barrier" and steps < AHEAD and int(m[1]) > PANELS * (AHEAD - 1):
                    break
            elif c.op == "s_barrier":
                steps = min(steps + 1, AHEAD)
                barriers.add(c.addr)
                if len(since) < need or left > since[0]:
                    found.add(c.addr)
            if c.op == "s_endpgm":
                break
            if c.target in at and c.op.startswith(("s_cbranch", "s_branch")):
                todo.append((at[c.target], since, left, steps))
                if c.op.startswith("s_branch"):
                    break
                todo.append((i + 1, since, left, steps))
                break
            i += 1
    return barriers, sorted(found)


def _product_kernels(tmp_path):
    K.lib()
    kernels = {}
    for obj in _code_objects(K._LIB_PATH, str(tmp_path)):
        text = subprocess.run([f"{LLVM}/llvm-objdump", "-d", "--no-show-raw-insn", obj], check=True, capture_output=True,
                              text=True).stdout
        for m in re.finditer(r"^([0-9a-f]+) <(\S*%s\S*)>:\n((?:\t.*\n)+)" % KERNELS, text, re.M):
            kernels[m[2]] = parse(m[3].splitlines(), int(m[1], 16))
    return kernels


def test_no_hazard_in_the_product_kernels(tmp_path):
    kernels = _product_kernels(tmp_path)
    # grad_W_s: 3 tiles x order x type x add; grad_h_s: 4 tiles x order; grad_W_s of few tokens: order x type x add
    assert len(kernels) == 24 + 8 + 8
    for name, code in kernels.items():
        assert sum("ds_read_b64" in c.op for c in code) >= 2 * 2 * 4, name
        assert early_uses(code) == [], name
        if "grad_w_few" not in name:
            assert hazards(code) == [], name


def test_few_tokens_wait_for_their_stages(tmp_path):
    few = {name: code for name, code in _product_kernels(tmp_path).items() if "grad_w_few" in name}
    assert len(few) == 8
    for name, code in few.items():
        barriers, late = late_waits(code)
        assert barriers and late == [], name
        if "ELb1EEE" in name:                 # (adding: what it adds to is waited for with everything older, on top of the count)
            continue
        # a wait that leaves one operation more in flight, or a step with an operation less, is seen
        waits = [i for i, c in enumerate(code[:-1]) if c.op == "s_waitcnt" and code[i + 1].op == "s_barrier"]
        most = max(waits, key=lambda i: int(re.search(r"vmcnt\((\d+)\)", code[i].operands[0])[1]))
        n = int(re.search(r"vmcnt\((\d+)\)", code[most].operands[0])[1])
        assert late_waits(code[:most] + [code[most]._replace(operands=[f"vmcnt({n + 1})"])] + code[most + 1:])[1], name
        stores = [i for i, c in enumerate(code) if c.op.startswith("buffer_store")]
        store = next((i for i in stores if i > most), stores[-1])
        assert late_waits(code[:store] + [code[store]._replace(op="s_nop")] + code[store + 1:])[1], name


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
