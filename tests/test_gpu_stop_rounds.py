"""Stop at the first satisfying particle in batches of more tiles than the chip
holds at once, and in tiles of several particles: bit for bit against calls of
one iteration, with waypoints (whose moments stay in device memory) and frozen
grasps, at stops that fall inside a launch.  A stop at the first iteration,
found by the last tile, costs a few iterations, not a whole launch of them."""
import pytest

from paper_2411_11833_amd import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

NONE = 2 ** 31 - 1


def _adam(n):
    from paper_2411_11833_amd.binding import CtAdam
    return CtAdam(2e-3, 0.9, 0.999, 1e-8, 1.0 / n)


def _problem(K, waypoints, tau):
    """Only the position errors decide Eq. (3)."""
    prob = I.packing(0, 1, n_objects=K, n_obstacles=2, waypoints=waypoints)
    prob.tolerances = I.Tolerances(kin_pos=tau, kin_rot=4.0, grasp=9.0, place=9.0, jlim=9.0, coll=99.0,
                                   motion_coll=999.0)
    return prob


def _state(gp, n, seed):
    X, M, V = gp.empty(n), gp.empty(n), gp.empty(n)
    gp.seed_uniform(seed, X, M, V, n)
    cost, mask = torch.zeros(n, device="cuda"), torch.zeros(n, dtype=torch.uint8, device="cuda")
    return X, M, V, cost, mask, torch.full((1,), NONE, dtype=torch.int32, device="cuda")


def _worst(gp, X, n):
    """The largest position error of every particle."""
    _, T, _ = gp.cost(X, n, terms=True)
    K = gp.prob.skeleton.n_steps
    return torch.stack([T[11 * k + j, :n] for k in range(K) for j in (0, 2)]).max(0).values


def _tolerance(K, waypoints, n, split, at):
    """A tolerance that some particle meets at iteration `at` or the next one
    that lowers the smallest error, and none before."""
    from paper_2411_11833_amd.planner import GpuProblem, grasp_frozen
    gp = GpuProblem(_problem(K, waypoints, 0.0))
    gp.set_split(split)
    s, best = _state(gp, n, 11), float("inf")
    for t in range(120):
        w = _worst(gp, s[0], n).min().item()
        if t >= at and w < best:
            return w, t
        best = min(best, w)
        gp.optimize(*s[:3], n, t, 1, _adam(n), frozen=grasp_frozen(gp.prob))
    raise AssertionError("no iteration lowers the error")


@pytest.mark.parametrize("K,split,n,waypoints", [(6, 4, 3001, 0), (2, 1, 2003, 0), (6, 4, 2700, 2), (1, 4, 1500, 3)])
@pytest.mark.parametrize("at", [0, 1, 17, 66])
def test_stop_equals_single_iterations(K, split, n, waypoints, at):
    from paper_2411_11833_amd.planner import GpuProblem, grasp_frozen
    tau, f = _tolerance(K, waypoints, n, split, at)
    gp = GpuProblem(_problem(K, waypoints, tau))
    gp.set_split(split)
    fz = grasp_frozen(gp.prob)
    a, b = _state(gp, n, 11), _state(gp, n, 11)
    for t, c in ((0, 90), (90, 40)):
        gp.optimize(*a[:3], n, t, c, _adam(n), frozen=fz, cost=a[3], mask=a[4], first_sat=a[5], stop_at_first=True)
    for t in range(130):
        gp.optimize(*b[:3], n, t, 1, _adam(n), frozen=fz, cost=b[3], mask=b[4], first_sat=b[5], stop_at_first=True)
    torch.cuda.synchronize()
    assert int(a[5].item()) == f
    assert all(torch.equal(u, v) for u, v in zip(a, b))
    assert 0 < int(a[4].sum().item())


def test_an_early_stop_in_the_last_tile_is_cheap():
    from paper_2411_11833_amd.planner import GpuProblem
    n = 4 * 512 * 32   # four rounds of full tiles
    gp = GpuProblem(_problem(4, 0, 10.0))
    gp.set_split(1)
    s = _state(gp, n, 11)
    s[0][18, :n - 1] += 100.0   # one particle satisfies, in the tile that starts last; the others never will
    X0 = s[0].clone()

    def run(iters):
        times = []
        for _ in range(4):
            s[0].copy_(X0)
            s[1].zero_()
            s[2].zero_()
            s[5].fill_(NONE)
            torch.cuda.synchronize()
            torch.cuda._sleep(2000000)   # the launches are queued before the first one starts
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            gp.optimize(*s[:3], n, 0, iters, _adam(n), cost=s[3], mask=s[4], first_sat=s[5], stop_at_first=True)
            e1.record()
            e1.synchronize()
            assert int(s[5].item()) == 0 and int(s[4].sum().item()) == 1 and int(s[4][n - 1].item()) == 1
            times.append(e0.elapsed_time(e1))
        return min(times)

    one, many = run(1), run(64)
    print(f"1 iteration {one * 1e3:.0f} us, 64 iterations stopped at the first {many * 1e3:.0f} us")
    assert many <= 8 * one


def test_no_copies_of_a_large_state():
    """The handle of a solve does not hold as much memory again as its buffers."""
    from paper_2411_11833_amd.planner import GpuProblem
    gp = GpuProblem(_problem(6, 0, 0.0))
    n = 720000   # 1.01 GiB of copies
    a, b = _state(gp, n, 11), _state(gp, n, 11)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    gp.optimize(*a[:3], n, 0, 3, _adam(n), cost=a[3], mask=a[4], first_sat=a[5], stop_at_first=True)
    torch.cuda.synchronize()
    assert free - torch.cuda.mem_get_info()[0] < 64 << 20
    for t in range(3):
        gp.optimize(*b[:3], n, t, 1, _adam(n), cost=b[3], mask=b[4], first_sat=b[5], stop_at_first=True)
    torch.cuda.synchronize()
    assert all(torch.equal(u, v) for u, v in zip(a, b))
