"""A particle with a NaN coordinate: the collision terms of the configurations
that the coordinate enters are NaN (or, for a placement, whose height is known,
positive), so that neither Eq. (5)'s counts nor the per-step masks take them
for satisfied.  One NaN at each coordinate in turn, against the terms of the
FP64 oracle; tiles with and without empty columns."""
import numpy as np
import pytest

import oracle as O
from paper_2411_11833_amd import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

COLL = (8, 9, 10)   # of a step's 11 terms: grasp and place configuration, placed object


@pytest.mark.parametrize("copies", [1, 40])
@pytest.mark.parametrize("split", [1, 2, 4])
def test_nan_coordinate_satisfies_no_collision_term(split, copies):
    from paper_2411_11833_amd.planner import GpuProblem
    prob = I.packing(0, 1, n_objects=2, n_obstacles=3)
    gp = GpuProblem(prob)
    gp.set_split(split)
    n = gp.dim * copies
    d = np.arange(n) % gp.dim
    X = I.uniform_particles(prob, n, seed=9)
    X[np.arange(n), d] = np.nan
    Xd = gp.from_rows(X)
    _, T, mask = gp.cost(Xd, n, terms=True)
    _, G = gp.cost_grad(Xd, n)
    counts, _ = gp.feasibility(T, n)
    steps, held = gp.step_mask(T, n)
    torch.cuda.synchronize()
    got, want = gp.to_rows(T, n).cpu().numpy(), O.terms(prob, X.astype(np.float64))
    eps = prob.tolerances.coll
    for k in range(2):
        for j in COLL:
            c = 11 * k + j
            r = d - 21 * k
            own = np.isnan(want[:, c]) & (0 <= r) & (r < 21)   # the step's own coordinates
            assert own.any()
            placed = own & (r >= 18)
            assert np.all(np.isnan(got[own & ~placed, c]))
            assert not np.any(got[placed, c] <= eps)
            assert int(counts[c]) == int((got[:, c] <= eps).sum()) <= n - own.sum()
            assert not steps[k].cpu().numpy()[:n][own].any()
    g = gp.to_rows(G, n).cpu().numpy()
    assert not np.isfinite(g[d % 21 < 18]).all(1).any()   # no joint or grasp NaN passes for a gradient
    assert not mask.any() and np.all(held.cpu().numpy() < gp.n_constraint)
