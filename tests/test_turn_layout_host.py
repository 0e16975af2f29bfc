"""LDS layout of the M2L with whole vectors per lane: every array aligned to what it is read by, and inside the
bytes that a launch asks for, at every order, type, number of potentials and of targets."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1201_5430_amd", "csrc")

SOURCE = r"""
#include "lhf_m2l_turn.h"
using namespace lhf;
template <typename T, int P, int NPOT>
constexpr bool ok()
{
    for (int ns = 1; ns <= 60; ns++) {
        const tn::Lds o = tn::lds<T, P, NPOT>(ns);
        if (o.trl % (2 * sizeof(T)) || o.acc % sizeof(double) || o.esrc % sizeof(int) || o.sxyz % sizeof(int) ||
            o.ssys % sizeof(int) || o.cnt % sizeof(int) || o.ecode % sizeof(uint16_t))
            return false;
        if (o.end > tn::fixed_bytes<T, P, NPOT>() + ns * tn::slot_bytes<T, P, NPOT>()) return false;
    }
    return true;
}
#define CHECK(T, P) static_assert(ok<T, P, 1>() && ok<T, P, 2>(), #T " " #P);
"""


def test_layout(tmp_path):
    if not shutil.which("hipcc"):
        pytest.skip("needs hipcc")
    src = tmp_path / "layout.hip"
    src.write_text(SOURCE + "".join(f"CHECK({t}, {p})\n" for t, top in (("double", 13), ("float", 17))
                                    for p in range(7, top)))
    r = subprocess.run(["hipcc", "-std=c++17", "--cuda-host-only", "-fsyntax-only", "--offload-arch=gfx950", "-I", CSRC,
                        "-fconstexpr-steps=100000000", str(src)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
