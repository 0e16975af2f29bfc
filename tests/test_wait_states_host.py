"""Wait states of the row kernels along every path: a register that the vector unit wrote may be read by a row
broadcast or a lane exchange only two wait states later, also over a branch and round a loop's back edge.  (The
compiler's own check does not look into the inline multiplications; straight-line reading is tested beside the
kernels' other host checks.)  The built objects' code is read back."""
import glob
import os
import re
import shutil

import pytest

import test_turn_host as host


def _functions(text):
    """[(address, opcode, operands, branch target or None)] of every function of a disassembly"""
    out, base = [], 0
    for line in text.splitlines():
        m = re.match(r"^([0-9a-f]+) <.*>:", line)
        if m:
            base = int(m[1], 16)
            out.append([])
            continue
        m = re.match(r"^\s+(\S+)\s*(.*?)\s*//\s*([0-9A-F]+):[ 0-9A-F]*(?:<.*?(?:\+0x([0-9a-f]+))?>)?$", line)
        if m and out:
            to = base + int(m[4] or "0", 16) if "branch" in m[1] else None
            out[-1].append((int(m[3], 16), m[1], [o.strip() for o in m[2].split(",")], to))
    return out


def _written(ins):
    op, ops = ins[1], ins[2]
    if not op.startswith("v_") or op.startswith(("v_cmp", "v_readlane", "v_readfirst")):
        return set()
    return host._regs(ops[0].split()[0]) | (host._regs(ops[1].split()[0]) if "swap" in op else set())


def _missing(code):
    """(reads that need wait states, those without them) of one function"""
    at = {ins[0]: i for i, ins in enumerate(code)}
    before = [[] for _ in code]
    for i, (_, op, _, to) in enumerate(code):
        if to is not None:
            before[at[to]].append(i)
        if op.startswith("s_setpc"):  # a far jump: three scalar instructions form the address, wait states enough
            assert all(code[i - k][1].startswith("s_") for k in (1, 2, 3)), code[i]
        elif op not in ("s_branch", "s_endpgm") and i + 1 < len(code):
            before[i + 1].append(i)

    def late(i, regs, n):
        return any(_written(code[j]) & regs or
                   (n > (k := int(code[j][2][0], 0) + 1 if code[j][1] == "s_nop" else 1) and late(j, regs, n - k))
                   for j in before[i])

    seen, bad = 0, []
    for i, (_, op, ops, _) in enumerate(code):
        row = op.startswith("v_") and ("dpp" in op or any("row_" in o or "quad_perm" in o for o in ops))
        lanes = op.startswith("v_permlane")
        if row or lanes:
            seen += 1
            regs = host._regs(ops[1].split()[0]) | (host._regs(ops[0]) if lanes else set())
            if late(i, regs, 2):
                bad.append(code[i])
    return seen, bad


LOOP = """
0000000000000100 <k>:
	v_mov_b32_e32 v1, v2                                       // 000000000100: 7E020302
	s_nop 1                                                    // 000000000104: BF800001
	v_fmac_f64_dpp v[4:5], v[0:1], v[2:3] row_newbcast:0       // 000000000108: 08040400 FF010000
	s_cbranch_scc1 65533                                       // 000000000110: BF85FFFD <k+0x{:x}>
	s_endpgm                                                   // 000000000114: BF810000
"""


def test_the_reading_follows_branches():
    assert _missing(_functions(LOOP.format(4))[0]) == (1, [])
    # round the loop: v[4:5] is written by the multiplication, and read a branch later
    text = LOOP.replace("v[0:1], v[2:3]", "v[4:5], v[2:3]")
    assert len(_missing(_functions(text.format(8))[0])[1]) == 1
    assert _missing(_functions(text.format(4))[0]) == (1, [])


@pytest.mark.parametrize("kind", ["m2l_rows", "mm_rows"])
def test_built_kernels(kind, tmp_path):
    objs = sorted(glob.glob(os.path.join(host.CSRC, f"lhf_{kind}_*.o")))
    if not objs or not shutil.which(f"{host.LLVM}/llvm-objdump"):
        pytest.skip("needs the built objects and the LLVM tools")
    for o in objs:
        for code in _functions(host._disassemble(o, tmp_path)):
            seen, bad = _missing(code)
            assert seen > 100 and not bad, (o, seen, bad[:3])
