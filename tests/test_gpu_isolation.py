"""Systems of one plan do not see each other, also where a system's strengths are not finite: the boxes of
two systems share the M2L's tiles, its batches and, in the kernels with a vector split over rows, the LDS that
the odd orders' last pair reads one entry of beside its angles.

A system with non-finite strengths ends in the corner of its cube that lies last along the curve, so its boxes
take the first slots of a tile; the system behind it has three boxes whose translations (directions (0, 1, 3)
and (1, 0, 3)) come last in the tile's list.

Bars: the same plan with the other systems at rest differs by the order of the sums alone (FP64 1e-13 in L2 and
1e-12 element-wise, FP32 2e-6 and 1e-5)."""
import numpy as np
import pytest

from parity_util import check, check32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bad", [np.inf, np.nan])
@pytest.mark.parametrize("prec,p", [(0, 6), (0, 9), (0, 12), (0, 13), (0, 16), (0, 21), (0, 23), (1, 10), (1, 15)])
def test_non_finite_system(prec, p, bad):
    import torch
    import paper_1201_5430_amd as L
    rng = np.random.default_rng(40 + p)
    dt = torch.float64 if prec == 0 else torch.float32
    x, off, ok = [], [0], []
    for k in range(24):
        x.append(rng.uniform(0, 1, (260, 3)))
        corner = np.array([[0, 0, 0], [1, 0, 3], [0, 1, 3]]) / 8.0
        x.append(np.repeat(corner, 2, axis=0) + rng.uniform(0.01, 0.11, (6, 3)))
        off += [off[-1] + 260, off[-1] + 266]
        ok += [False] * 260 + [True] * 6
    x, ok = np.concatenate(x), np.array(ok)
    w = rng.normal(size=x.shape)
    xt = torch.from_numpy(x).to("cuda", dt)
    plan = L.Plan(xt, [0.01] * 48, p=p, depth=3, precision=prec, offsets=np.array(off))
    out = []
    for other in (0.0, bad):
        v, s = plan.execute(torch.from_numpy(np.where(ok[:, None], w, other)).to("cuda", dt))
        torch.cuda.synchronize()
        out.append((v.double().cpu().numpy()[ok], s.double().cpu().numpy()[ok]))
    plan.close()
    if prec == 0:
        check(*out[1], *out[0], l2=1e-13, mx=1e-12, label=f"isolation p={p}:")
    else:
        check32(*out[1], *out[0], label=f"isolation FP32 p={p}:")
