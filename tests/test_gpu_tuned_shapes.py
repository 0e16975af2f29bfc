"""The shapes that lhf_plan_autotune keeps are not slower than the built-in ones, in the launches that an
execute makes (all levels' M2L in one), and within what the running kernel holds."""
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", [16, 23])
def test_tuned_is_not_slower(p):
    import torch
    import paper_1201_5430_amd as L
    n = 500000
    x, w = workloads.vortex_ring(n, 801)
    xt, wt = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    plan = L.Plan(xt, workloads.core_radius(n), p=p, depth=8, max_per_leaf=64)

    def times():
        plan.execute(wt)
        best = {}
        for _ in range(5):
            plan.profile_begin(1)
            plan.execute(wt)
            ph = plan.profile_end()[0]
            best = {k: min(best.get(k, 1e9), ph[k]) for k in ("m2l", "p2p")}
        return best

    before = times()
    shapes = plan.autotune(wt)
    after = times()
    plan.close()
    print(f"p={p}: built-in {before}, tuned {after} with {shapes}", flush=True)
    # 8%: between what repeated runs of one shape differ by (2%) and what tuning level by level lost (13%, 31%)
    assert after["m2l"] <= 1.08 * before["m2l"] and after["p2p"] <= 1.08 * before["p2p"], (before, after, shapes)
