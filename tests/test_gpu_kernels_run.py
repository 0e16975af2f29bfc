"""lhf_plan_kernels names the kernels that run (m2l_runs, mm_runs of stats()), for every way of choosing them."""
import pytest

import workloads

F64, F32 = 0, 1
AUTO, HALF, GENERIC, QUARTER = 0, 1, 5, 6  # m2l_kernel
MM_HALF, MM_GENERIC, MM_QUARTER = 1, 2, 3


def test_null_plan():
    import paper_1201_5430_amd as L
    assert L.load().lhf_plan_kernels(None, None, None) == -1


@pytest.mark.gpu
@pytest.mark.parametrize("prec,p,kw,m2l,mm", [
    (F64, 6, {}, "tile", "generic"),
    (F64, 7, {}, "turn", "rows"),
    (F64, 12, {}, "turn", "rows"),
    (F64, 13, {}, "rows", "rows"),
    (F64, 23, {}, "rows", "rows"),
    (F32, 10, {}, "turn", "rows"),
    (F32, 16, {}, "turn", "rows"),
    (F64, 12, dict(deterministic=True), "mfma", "half"),
    (F64, 13, dict(deterministic=True), "generic", "generic"),
    (F64, 9, dict(depth=9), "generic", "generic"),
    (F64, 12, dict(m2l_kernel=HALF), "half", "half"),
    (F64, 23, dict(m2l_kernel=QUARTER), "quarter", "quarter"),
    (F64, 12, dict(m2l_kernel=GENERIC), "generic", "half"),
    (F64, 12, dict(mm_kernel=MM_HALF), "turn", "half"),
    (F64, 20, dict(mm_kernel=MM_QUARTER), "rows", "quarter"),
    (F32, 11, dict(mm_kernel=MM_GENERIC), "turn", "generic"),
])
def test_names(prec, p, kw, m2l, mm):
    import torch
    import paper_1201_5430_amd as L
    x, _ = workloads.uniform_cube(400, 5)
    kw = dict(dict(depth=3), **kw)
    xt = torch.from_numpy(x).to("cuda", torch.float64 if prec == F64 else torch.float32)
    plan = L.Plan(xt, 0.01, p=p, precision=prec, **kw)
    st = plan.stats()
    plan.close()
    assert (st["m2l_runs"], st["mm_runs"]) == (m2l, mm)
