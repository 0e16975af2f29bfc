"""The file of tuned shapes names the M2L kernel that they were measured with: plans of one workload with other
kernels, and entries without a name, do not share them; and a plan reports the shapes that run."""
import json

import pytest

import workloads

pytestmark = pytest.mark.gpu


def _plan(x, **kw):
    import paper_1201_5430_amd as L
    return L.Plan(x, workloads.core_radius(len(x)), p=23, depth=6, max_per_leaf=64, **kw)


def test_kernels_do_not_share_shapes(tmp_path):
    import torch
    import paper_1201_5430_amd as L
    x, w = workloads.vortex_ring(6000, 811)
    x, w = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    path = tmp_path / "shapes.json"
    path.write_text('[\n {"key": "gfx950/fp64/p23/adaptive/d6/n6000", "m2l_tile": [0, 0, 6, 6, 6, 6, 6, 0, 0], '
                    '"p2p_tile": 64}\n]\n')
    got = {}
    for name, kw in (("ROWS", {}), ("GENERIC", dict(deterministic=True)), ("QUARTER", dict(m2l_kernel=L.M2L_QUARTER))):
        plan = _plan(x, **kw)
        got[name] = plan.autotune(w, cache_path=str(path))
        assert got[name] == plan.get_shapes()
        plan.close()
    entries = json.loads(path.read_text())
    assert len(entries) == 4 and entries[0]["key"].endswith("/n6000")  # the nameless one stays in the file
    assert [e["key"].rsplit("/", 1)[1] for e in entries[1:]] == ["ROWS", "GENERIC", "QUARTER"]
    assert max(got["ROWS"]["m2l_tile"]) <= 5 and max(got["GENERIC"]["m2l_tile"]) == 0
    for e in entries[1:]:
        assert got[e["key"].rsplit("/", 1)[1]] == {k: e[k] for k in ("m2l_tile", "p2p_tile")}
    plan = _plan(x)  # read back
    assert plan.autotune(w, cache_path=str(path)) == got["ROWS"] and len(json.loads(path.read_text())) == 4
    plan.close()


def test_shapes_read_back_are_those_that_run():
    import torch
    import paper_1201_5430_amd as L
    x, _ = workloads.vortex_ring(6000, 811)
    x = torch.from_numpy(x).cuda()
    ask = dict(m2l_tile=[0, 0, 6, 6, 4, 6, 1, 0, 0], p2p_tile=64)
    for kw, mx in (({}, 5), (dict(m2l_kernel=L.M2L_QUARTER), 6)):
        plan = _plan(x, **kw)
        plan.set_shapes(ask)
        assert plan.get_shapes() == dict(ask, m2l_tile=[min(t, mx) for t in ask["m2l_tile"]])
        plan.close()
