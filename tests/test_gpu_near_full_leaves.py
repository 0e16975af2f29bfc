"""Near field of a uniform tree with few, full leaves: several workgroups share a leaf's targets.  Against the
oracle at leaf sizes around the chunks of 64 that are dealt out, and the time of a pair against that in a tree
with eight times the leaves: the work of 64 leaves has to spread over the chip as well.

Bars: those of the other comparisons with the oracle.  The pair's time may be 2.5 times that of the deeper tree
(with one workgroup a leaf it was 6.5 times)."""
import numpy as np
import pytest

from parity_util import check, check32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("full", [False, True], ids=["v s", "grad q"])
@pytest.mark.parametrize("c", [65, 127, 128, 129, 700])
def test_leaf_sizes(oracle, prec, full, c):
    import torch
    import paper_1201_5430_amd as L
    rng = np.random.default_rng(300 + c)
    # c elements in one leaf and its neighbour each, 96 or less in the others
    low = np.stack(np.meshgrid(*[np.arange(4)] * 3, indexing="ij"), -1).reshape(-1, 3) / 4.0
    num = np.where(np.arange(64) < 2, c, rng.integers(1, 97, 64))
    x = np.repeat(low, num, axis=0) + rng.uniform(0.001, 0.249, (num.sum(), 3))
    w, q, a = rng.normal(size=x.shape), rng.normal(size=len(x)), 0.02
    dt = torch.float64 if prec == 0 else torch.float32
    if prec:
        x, w, q = (u.astype(np.float32).astype(np.float64) for u in (x, w, q))
        a = float(np.float32(a))
    xt, wt, qt = (torch.from_numpy(u).to("cuda", dt) for u in (x, w, q))
    plan = L.Plan(xt, a, p=6, depth=2, precision=prec, grad=full)
    out = plan.execute(wt, what=2, q=qt if full else None, grad=full)
    again = plan.execute(wt, what=2, q=qt if full else None, grad=full)
    torch.cuda.synchronize()
    plan.close()
    assert all(torch.equal(u, v) for u, v in zip(out, again))
    ref = oracle.fmm(x, w, a, 6, 2, far=False, q=q if full else None, grad=full)
    out = [t.double().cpu().numpy() for t in out]
    (check if prec == 0 else check32)(out[0], out[1], ref[0], ref[1], label=f"full leaves c={c} prec={prec}:")


@pytest.mark.parametrize("prec", [0, 1])
def test_spread_over_the_chip(prec):
    import torch
    import paper_1201_5430_amd as L
    n = 65536
    dt = torch.float64 if prec == 0 else torch.float32
    rng = np.random.default_rng(310)
    x = torch.from_numpy(rng.uniform(0, 1, (n, 3))).to("cuda", dt)
    w = torch.from_numpy(rng.normal(size=(n, 3))).to("cuda", dt)
    pair = []
    for depth in (2, 3):
        plan = L.Plan(x, 0.5 * n ** (-1 / 3), p=6, depth=depth, precision=prec)
        pairs = plan.stats()["n_p2p_pairs"]
        plan.execute(w, what=2)
        best = float("inf")
        for _ in range(5):
            plan.profile_begin(1)
            plan.execute(w, what=2)
            best = min(best, plan.profile_end()[0]["p2p"])
        plan.close()
        pair.append(best * 1e9 / pairs)
    print(f"near field prec={prec}: {pair[0]:.2f} ps a pair in 64 leaves, {pair[1]:.2f} in 512", flush=True)
    assert pair[0] <= 2.5 * pair[1], pair
