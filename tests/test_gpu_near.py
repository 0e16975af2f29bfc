"""The near field alone against the oracle's, at the leaf sizes where the split of lanes over targets and
sources changes: a leaf of c elements takes them 1 to 64 at a time, and its sources pass through an index
table of 1,024 entries.  'few': one workgroup of four wavefronts a leaf; 'many': one wavefront a leaf, from
8,192 leaves on.  The core radii put the pairs on both sides of u = r^2 / (2 a^2) = 1 and of the cutoff.

Bars: those of the other comparisons with the oracle (FP64 1e-12 in L2 and 1e-11 element-wise, FP32 2e-6
and 1e-5): both sum the same pairs, and no pair loses more than a few units of rounding."""
import numpy as np
import pytest

from parity_util import check, check32

pytestmark = pytest.mark.gpu


def _points(c, many, seed):
    """c elements inside one leaf, the others spread over the cube"""
    rng = np.random.default_rng(seed)
    depth = 5 if many else 2
    h = 2.0 ** -depth
    x = rng.uniform(0, 1, (10500 if many else 700, 3))
    inside = ((x >= h) & (x < 2 * h)).all(axis=1)
    x = np.concatenate([x[~inside], h + h * rng.uniform(0.001, 0.999, (c, 3))])
    x = x[rng.permutation(len(x))]
    return x, rng.normal(size=x.shape), rng.normal(size=len(x)), depth


def _run(oracle, x, w, q, a, depth, prec, full):
    import torch
    import paper_1201_5430_amd as L
    dt = torch.float64 if prec == 0 else torch.float32
    if prec:
        x, w, q = (u.astype(np.float32).astype(np.float64) for u in (x, w, q))
        a = float(np.float32(a))
    xt, wt, qt = (torch.from_numpy(u).to("cuda", dt) for u in (x, w, q))
    plan = L.Plan(xt, a, p=6, depth=depth, precision=prec, grad=full)
    out = plan.execute(wt, what=2, q=qt if full else None, grad=full)
    torch.cuda.synchronize()
    plan.close()
    ref = oracle.fmm(x, w, a, 6, depth, far=False, q=q if full else None, grad=full)
    chk = check if prec == 0 else check32
    label = f"near n={len(x)} prec={prec} full={full}"
    out = [t.double().cpu().numpy() for t in out]
    chk(out[0], out[1], ref[0], ref[1], label=label)
    if full:
        chk(out[2], out[2], ref[2], ref[2], label=label + " grad v")


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("many", [False, True], ids=["few", "many"])
@pytest.mark.parametrize("c", [1, 2, 15, 17, 33, 63, 64, 65, 130, 1100])
def test_leaf_sizes(oracle, prec, many, c):
    x, w, q, depth = _points(c, many, 40 + c)
    _run(oracle, x, w, q, 0.5 * len(x) ** (-1 / 3), depth, prec, full=(c % 2 == 1))


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("a", [1e-3, 0.03, 0.3, 3.0])
def test_core_radii(oracle, prec, a):
    x, w, q, depth = _points(60, False, 77)
    _run(oracle, x, w, q, a, depth, prec, full=True)
