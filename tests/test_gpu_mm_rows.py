"""M2M and L2L by quarter turns (with the default kernels from p = 7 on): every order built, in both
precisions, against the generic per-box kernels with the same M2L, on uniform, adaptive and multi-system
trees, with boxes of one to eight children, and for the scalar FMM; and the compiled kernels' wait states.

Bars: the kernels differ by rounding alone, those of the M2L's comparison (FP64 1e-13 in L2 and 1e-12
element-wise, FP32 2e-6 and 1e-5)."""
import glob
import os
import shutil

import numpy as np
import pytest

import test_turn_host as wait
import workloads
from parity_util import check, check32

ORDERS = [(0, p) for p in range(7, 25)] + [(1, p) for p in range(7, 17)]


def _pair(x, w, a, p, prec, **kw):
    import torch
    import paper_1201_5430_amd as L
    dt = torch.float64 if prec == 0 else torch.float32
    xt, wt = torch.from_numpy(x).to("cuda", dt), torch.from_numpy(w).to("cuda", dt)
    out = []
    for kernel in (L.MM_AUTO, L.MM_GENERIC):
        plan = L.Plan(xt, a, p=p, precision=prec, mm_kernel=kernel, **kw)
        v, s = plan.execute(wt, what=1)
        torch.cuda.synchronize()
        out.append((v.double().cpu().numpy(), s.double().cpu().numpy()))
        plan.close()
    label = f"mm rows n={len(x)} prec {prec} p={p}:"
    if prec == 0:
        check(*out[0], *out[1], l2=1e-13, mx=1e-12, label=label)
    else:
        check32(*out[0], *out[1], label=label)


@pytest.mark.gpu
@pytest.mark.parametrize("prec,p", ORDERS)
def test_uniform(prec, p):
    x, w = workloads.uniform_cube(2500, 700 + p)
    _pair(x, w, workloads.core_radius(2500), p, prec, depth=4)


@pytest.mark.gpu
@pytest.mark.parametrize("prec,p", [(0, 9), (0, 12), (0, 16), (0, 17), (0, 24), (1, 7), (1, 16)])
def test_adaptive(prec, p):
    x, w = workloads.vortex_ring(9000, 730 + p)
    _pair(x, w, workloads.core_radius(9000), p, prec, depth=7, max_per_leaf=12)


@pytest.mark.gpu
@pytest.mark.parametrize("prec,p", [(0, 8), (0, 13), (1, 11)])
@pytest.mark.parametrize("n", [3, 70])
def test_few_boxes(prec, p, n):
    x, w = workloads.uniform_cube(n, 750 + n)
    _pair(x, w, 0.01, p, prec, depth=4)


@pytest.mark.gpu
@pytest.mark.parametrize("prec,p", [(0, 11), (0, 18), (1, 10)])
def test_several_systems(prec, p):
    n = [900, 1, 40, 1300]
    x = np.concatenate([workloads.uniform_cube(k, 760 + k)[0] for k in n])
    w = np.concatenate([workloads.uniform_cube(k, 760 + k)[1] for k in n])
    _pair(x, w, [0.02] * len(n), p, prec, depth=4, offsets=np.concatenate([[0], np.cumsum(n)]))


def test_wait_states(tmp_path):
    objs = sorted(glob.glob(os.path.join(wait.CSRC, "lhf_mm_rows_*.o")))
    if not objs or not shutil.which(f"{wait.LLVM}/llvm-objdump"):
        pytest.skip("needs the built objects and the LLVM tools")
    for o in objs:
        seen, bad = wait._missing_waits(wait._disassemble(o, tmp_path))
        # both kernels turn four times, order n with (n // 2 + 1)^2 multiplications
        order = int(o[:-2].rsplit("_", 1)[1])
        assert seen >= 8 * sum((n // 2 + 1) ** 2 for n in range(order)), o
        assert not bad, (o, bad[:3])
