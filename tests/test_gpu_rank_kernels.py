"""Per-step masks and the feasibility counts of Eq. (5): several waves share a
particle's steps, and small products of constraints and particles take one
launch.  Row counts at the edges of a wave, of the counting loop (512) and of
the launch rule (2^17 terms), with waypoint and self-collision terms, NaN and
infinite terms and terms equal to their tolerance, against NumPy (whole
numbers: exact)."""
import numpy as np
import pytest

from paper_2411_11833_amd import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("K,waypoints,self_collision", [(1, 0, 0), (2, 3, 1), (4, 0, 1), (5, 2, 0), (6, 1, 1)])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 511, 513, 1500, 2048, 13000])
def test_masks_and_counts_match_numpy(K, waypoints, self_collision, n):
    import oracle as O
    from paper_2411_11833_amd.planner import GpuProblem
    prob = I.packing(3, 1, n_objects=K, n_obstacles=2)
    prob.skeleton.waypoints = waypoints
    prob.skeleton.self_collision = self_collision
    gp = GpuProblem(prob)
    eps = np.asarray(O.tolerance_vector(prob), dtype=np.float32)[:gp.n_constraint]
    rng = np.random.default_rng(n + K)
    t = (rng.uniform(0, 2, (gp.n_terms, n)) ** 4 * 0.05).astype(np.float32)
    t[rng.random(t.shape) < 0.6] = 0
    c = gp.n_constraint
    at = rng.random((c, n)) < 0.05
    t[:c][at] = np.broadcast_to(eps[:, None], (c, n))[at]
    t[rng.random(t.shape) < 0.02] = np.nan
    t[rng.random(t.shape) < 0.02] = np.inf
    t[c - 1] = np.inf   # one constraint that no particle meets: the penalty
    T = gp.empty(n, rows=gp.n_terms)
    T.fill_(-1.0)       # the padding would count as satisfied
    T[:, :n] = torch.from_numpy(t).cuda()
    ok = t[:c] <= eps[:, None]
    steps, count = gp.step_mask(T, n)
    counts, H = gp.feasibility(T, n)
    torch.cuda.synchronize()
    want = np.stack([ok[11 * k: 11 * (k + 1)].all(0) for k in range(K)])
    assert np.array_equal(steps[:, :n].cpu().numpy(), want.astype(np.uint8))
    assert np.array_equal(count.cpu().numpy(), ok.sum(0))
    assert np.array_equal(counts.cpu().numpy(), ok.sum(1))
    h = np.where(ok.sum(1) > 0, ok.sum(1), -n).astype(np.float64).sum() / c
    assert abs(float(H.item()) - h) <= abs(h) * 2.0 ** -23
