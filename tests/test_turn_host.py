"""Host checks of the M2L by quarter turns: the factorisation of the rotation about y and its zero pattern
(against the exponential of the generator), and the compiled kernels' wait states.

The kernels for rows multiply by inline assembly with row broadcasts, which the compiler's own check for
missing wait states does not look into: a register written by the vector unit may be read by a row
broadcast or a lane exchange only after two other wait states.  The built objects are read back for that."""
import glob
import math
import os
import re
import shutil
import subprocess

import numpy as np
import pytest
from scipy.linalg import expm

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1201_5430_amd", "csrc")
LLVM = "/opt/rocm/llvm/bin"


def _gen(n):
    """generator of rotations about y in the orthonormal basis, rows and columns m = -n .. n"""
    def g(m, mp):
        if mp == m - 1:
            return (0.5 if m >= 1 else -0.5) * math.sqrt((n + m) * (n - m + 1)) if m else -0.5 * math.sqrt(n * (n + 1))
        if mp == m + 1:
            return (0.5 if m < 0 else -0.5) * math.sqrt((n - m) * (n + m + 1)) if m else -0.5 * math.sqrt(n * (n + 1))
        return 0.0
    return np.array([[g(m, mp) for mp in range(-n, n + 1)] for m in range(-n, n + 1)])


def _b(n, th):
    """rotation by th on [Re 0 .. n | Im 1 .. n]"""
    E = expm(-th * _gen(n))
    c = lambda m: math.sqrt(2.0) if m else 1.0
    M = np.zeros((2 * n + 1, 2 * n + 1))
    for mp in range(n + 1):
        for m in range(n + 1):
            M[mp, m] = (E[m + n, mp + n] + (E[-m + n, mp + n] if m else 0.0)) * c(mp) / c(m)
            if m and mp:
                M[n + mp, n + m] = E[m + n, mp + n] - E[-m + n, mp + n]
    return M


def _z(n, ph):
    M = np.zeros((2 * n + 1, 2 * n + 1))
    M[0, 0] = 1.0
    for m in range(1, n + 1):
        M[m, m] = M[n + m, n + m] = math.cos(m * ph)
        M[m, n + m], M[n + m, m] = -math.sin(m * ph), math.sin(m * ph)
    return M


@pytest.mark.parametrize("n", [1, 2, 5, 12, 23])
def test_factorisation_and_zeros(n):
    h = math.pi / 2
    Y = _b(n, h)
    for th in (0.3, 1.1, 2.7):
        assert np.abs(_z(n, h) @ Y @ _z(n, math.pi + th) @ Y @ _z(n, h) - _b(n, th)).max() < 1e-12
    for mp in range(n + 1):
        for m in range(n + 1):
            if (m + mp + n) % 2:
                assert abs(Y[mp, m]) < 1e-13
            elif m and mp:
                assert abs(Y[n + mp, n + m]) < 1e-13


def _disassemble(obj, tmp):
    fb, co = str(tmp / "x.fb"), str(tmp / "x.co")
    subprocess.run([f"{LLVM}/llvm-objcopy", f"--dump-section=.hip_fatbin={fb}", obj], check=True)
    lst = subprocess.run([f"{LLVM}/clang-offload-bundler", "--list", "--type=o", f"--input={fb}"], check=True,
                         capture_output=True, text=True).stdout
    tgt = next(t for t in lst.split() if "gfx950" in t)
    subprocess.run([f"{LLVM}/clang-offload-bundler", "--unbundle", "--type=o", f"--targets={tgt}", f"--input={fb}",
                    f"--output={co}"], check=True)
    return subprocess.run([f"{LLVM}/llvm-objdump", "-d", "--no-show-raw-insn", "--mcpu=gfx950", co], check=True,
                          capture_output=True, text=True).stdout


def _regs(op):
    m = re.match(r"v\[(\d+):(\d+)\]", op)
    if m:
        return set(range(int(m[1]), int(m[2]) + 1))
    m = re.match(r"v(\d+)", op)
    return {int(m[1])} if m else set()


def _missing_waits(text):
    bad, seen, hist = [], 0, []
    for line in text.splitlines():
        if re.match(r"^[0-9a-f]+ <", line):
            hist = []
            continue
        m = re.match(r"^\s+(\S+)\s*(.*?)(?:\s*//.*)?$", line)
        if not m:
            continue
        op, ops = m[1], [o.strip() for o in m[2].split(",")]
        recent = set().union(*hist[-2:]) if hist else set()
        wrote = set()
        if op.startswith("v_"):
            if "dpp" in op or "row_" in m[2] or "quad_perm" in m[2]:
                seen += 1
                if _regs(ops[1].split()[0]) & recent:
                    bad.append(line.strip())
            if "permlane" in op:
                if (_regs(ops[0]) | _regs(ops[1].split()[0])) & recent:
                    bad.append(line.strip())
                wrote |= _regs(ops[1].split()[0])
            if not op.startswith(("v_cmp", "v_readlane", "v_readfirst")):
                wrote |= _regs(ops[0].split()[0])
        hist += [set()] * (int(ops[0], 0) + 1) if op == "s_nop" else [wrote]
        hist = hist[-4:]
    return seen, bad


def test_wait_states_of_the_row_kernels(tmp_path):
    objs = sorted(glob.glob(os.path.join(CSRC, "lhf_m2l_rows_*.o")))
    if not objs or not shutil.which(f"{LLVM}/llvm-objdump"):
        pytest.skip("needs the built objects and the LLVM tools")
    for o in objs:
        seen, bad = _missing_waits(_disassemble(o, tmp_path))
        assert seen > 1000, o
        assert not bad, (o, bad[:3])
