"""The M2L by quarter turns (the default from p = 7 on): every order built, in both precisions, against
the generic per-box kernel on the same tree, on uniform, adaptive and multi-system trees, with few boxes
and for the scalar FMM.

Bars: the two kernels differ by rounding alone.  FP64: 1e-13 (L2) and 1e-12 (largest element against the
largest magnitude), the bars of the other kernel-against-kernel comparisons.  FP32: 2e-6 and 1e-5, the bars
of the FP32 paths."""
import numpy as np
import pytest

import workloads
from parity_util import check, check32

pytestmark = pytest.mark.gpu


def _pair(x, w, a, p, prec, **kw):
    import torch
    import paper_1201_5430_amd as L
    dt = torch.float64 if prec == 0 else torch.float32
    xt, wt = torch.from_numpy(x).to("cuda", dt), torch.from_numpy(w).to("cuda", dt)
    out = []
    for kernel in (L.M2L_AUTO, L.M2L_GENERIC):
        plan = L.Plan(xt, a, p=p, precision=prec, m2l_kernel=kernel, **kw)
        v, s = plan.execute(wt)
        torch.cuda.synchronize()
        out.append((v.double().cpu().numpy(), s.double().cpu().numpy()))
        plan.close()
    return out


def _cmp(prec, a, b, label):
    if prec == 0:
        check(*a, *b, l2=1e-13, mx=1e-12, label=label)
    else:
        check32(*a, *b, label=label)


@pytest.mark.parametrize("prec,p", [(0, p) for p in range(7, 25)] + [(1, p) for p in range(7, 17)])
def test_uniform(prec, p):
    x, w = workloads.uniform_cube(2500, 900 + p)
    a, b = _pair(x, w, workloads.core_radius(2500), p, prec, depth=4)
    _cmp(prec, a, b, f"turn uniform prec {prec} p={p}:")


@pytest.mark.parametrize("prec,p", [(0, 9), (0, 12), (0, 13), (0, 19), (1, 11), (1, 16)])
def test_adaptive(prec, p):
    x, w = workloads.vortex_ring(9000, 930 + p)
    a, b = _pair(x, w, workloads.core_radius(9000), p, prec, depth=7, max_per_leaf=12)
    _cmp(prec, a, b, f"turn ring prec {prec} p={p}:")


@pytest.mark.parametrize("prec,p", [(0, 7), (0, 14), (1, 9)])
@pytest.mark.parametrize("n", [2, 65])
def test_few_boxes(prec, p, n):
    # less than one batch of translations, and a box or two per tile
    x, w = workloads.uniform_cube(n, 950 + n)
    a, b = _pair(x, w, 0.01, p, prec, depth=2)
    _cmp(prec, a, b, f"turn n={n} prec {prec} p={p}:")


@pytest.mark.parametrize("p", [9, 15])
def test_systems(p):
    rng = np.random.default_rng(960 + p)
    off = np.array([0, 300, 300, 1500, 1501, 2600])
    x = rng.uniform(0, 1, (2600, 3))
    w = rng.normal(size=(2600, 3))
    a, b = _pair(x, w, 0.02, p, 0, depth=3, offsets=off)
    _cmp(0, a, b, f"turn systems p={p}:")


@pytest.mark.parametrize("prec,p", [(0, 7), (0, 11), (0, 14), (0, 21), (1, 9), (1, 14)])
def test_scalar(prec, p):
    import torch
    import paper_1201_5430_amd as L
    dt = torch.float64 if prec == 0 else torch.float32
    rng = np.random.default_rng(970 + p)
    xt = torch.from_numpy(rng.uniform(0, 1, (3000, 3))).to("cuda", dt)
    q = torch.from_numpy(rng.normal(size=3000)).to("cuda", dt)
    out = []
    for kernel in (L.M2L_AUTO, L.M2L_GENERIC):
        plan = L.Plan(xt, 0.0, p=p, depth=4, precision=prec, m2l_kernel=kernel)
        phi, g = plan.execute_scalar(q)
        torch.cuda.synchronize()
        out.append((phi.double().cpu().numpy()[:, None], g.double().cpu().numpy()))
        plan.close()
    _cmp(prec, out[0], out[1], f"turn scalar prec {prec} p={p}:")


def test_noalloc_without_room_for_the_box_maps():
    # depth 8: the box maps of levels 2..8 and the copy of the sources do not fit the fixed array beside
    # this plan; the evaluation takes the kernel that needs neither
    import torch
    import paper_1201_5430_amd as L
    n = 13000
    x, w = workloads.uniform_cube(n, 980)
    xt, wt = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    a = workloads.core_radius(n)
    v, s = L.evaluate_noalloc(xt, wt, a, p=9, depth=8)
    plan = L.Plan(xt, a, p=9, depth=8, m2l_kernel=L.M2L_GENERIC)
    v2, s2 = plan.execute(wt)
    torch.cuda.synchronize()
    plan.close()
    check(v.cpu().numpy(), s.cpu().numpy(), v2.cpu().numpy(), s2.cpu().numpy(), l2=1e-13, mx=1e-12, label="noalloc:")
