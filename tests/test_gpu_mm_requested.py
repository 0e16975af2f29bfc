"""M2M and L2L kernels asked for by name, beside the M2L by quarter turns (the L2L adds to what the M2L of all
levels wrote) and beside an M2L of their own split (it writes before the M2L adds), against the generic per-box
shifts with the same M2L, on a uniform and an adaptive tree.

Bars: those of the other kernel-against-kernel comparisons (FP64 1e-13 in L2 and 1e-12 element-wise, FP32 2e-6
and 1e-5)."""
import numpy as np
import pytest

import workloads
from parity_util import check, check32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("adaptive", [False, True], ids=["uniform", "ring"])
@pytest.mark.parametrize("own", [False, True], ids=["quarter turns", "own M2L"])
@pytest.mark.parametrize("prec,p", [(0, 8), (0, 10), (0, 12), (0, 16), (0, 20), (0, 22), (0, 23), (0, 24), (1, 8), (1, 10),
                                    (1, 12), (1, 16)])
def test_requested(prec, p, own, adaptive):
    import torch
    import paper_1201_5430_amd as L
    half = p <= 16
    x, w = workloads.vortex_ring(9000, 600 + p) if adaptive else workloads.uniform_cube(2500, 600 + p)
    kw = dict(depth=7, max_per_leaf=12) if adaptive else dict(depth=4)
    if own:
        kw["m2l_kernel"] = L.M2L_HALF if half else L.M2L_QUARTER
    dt = torch.float64 if prec == 0 else torch.float32
    xt, wt = torch.from_numpy(x).to("cuda", dt), torch.from_numpy(w).to("cuda", dt)
    out, runs = [], []
    for mm in (L.MM_HALF if half else L.MM_QUARTER, L.MM_GENERIC):
        plan = L.Plan(xt, workloads.core_radius(len(x)), p=p, precision=prec, mm_kernel=mm, **kw)
        v, s = plan.execute(wt, what=1)
        torch.cuda.synchronize()
        out.append((v.double().cpu().numpy(), s.double().cpu().numpy()))
        st = plan.stats()
        runs.append((st["m2l_runs"], st["mm_runs"]))
        plan.close()
    name = "half" if half else "quarter"
    m2l = name if own else "rows" if prec == 0 and p > 12 else "turn"
    assert runs == [(m2l, name), (m2l, "generic")]
    label = f"{name} M2M/L2L prec {prec} p={p} beside {m2l}:"
    if prec == 0:
        check(*out[0], *out[1], l2=1e-13, mx=1e-12, label=label)
    else:
        check32(*out[0], *out[1], label=label)
