"""P2M by sums of strengths times harmonics: the far field alone against the oracle's, for leaves at the
edges of the kernel's chunks of elements (16 at low orders, 7 at FP64 p = 24), the lowest, an ordinary and
the highest order, with and without monopoles.

Bars: those of the other comparisons with the oracle (FP64 1e-12 in L2, 1e-11 element-wise; FP32 2e-6, 1e-5)."""
import numpy as np
import pytest

from parity_util import check, check32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,p", [(0, 2), (0, 8), (0, 24), (1, 3), (1, 16)])
@pytest.mark.parametrize("c,mono", [(1, False), (7, True), (8, False), (16, True), (17, False), (33, True)])
def test_chunk_edges(oracle, prec, p, c, mono):
    import torch
    import paper_1201_5430_amd as L
    rng = np.random.default_rng(900 + c)
    # every leaf of a depth-2 tree holds c elements, one leaf five more
    low = np.stack(np.meshgrid(*[np.arange(4)] * 3, indexing="ij"), -1).reshape(-1, 1, 3) / 4.0
    x = (low + rng.uniform(0.01, 0.24, (64, c, 3))).reshape(-1, 3)
    x = np.concatenate([x, rng.uniform(0.26, 0.49, (5, 3))])
    w, q, a = rng.normal(size=x.shape), rng.normal(size=len(x)), 0.01
    dt = torch.float64 if prec == 0 else torch.float32
    if prec:
        x, w, q = (u.astype(np.float32).astype(np.float64) for u in (x, w, q))
        a = float(np.float32(a))
    xt, wt, qt = (torch.from_numpy(u).to("cuda", dt) for u in (x, w, q))
    plan = L.Plan(xt, a, p=p, depth=2, precision=prec)
    out = plan.execute(wt, what=1, q=qt if mono else None)
    torch.cuda.synchronize()
    plan.close()
    ref = oracle.fmm(x, w, a, p, 2, near=False, q=q if mono else None)
    v, s = (t.double().cpu().numpy() for t in out[:2])
    (check if prec == 0 else check32)(v, s, ref[0], ref[1], label=f"p2m prec={prec} p={p} c={c} mono={mono}:")
