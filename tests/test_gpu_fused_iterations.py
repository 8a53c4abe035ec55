"""ct_optimize runs many iterations of a tile in one launch.  Checked bit for
bit against one launch per iteration (ct_step, or ct_optimize one iteration at
a time where the stop at the first satisfying particle is on): the launch
boundary at 64 iterations, ragged tiles, and stops that one tile finds while
the others have already run past it."""
import numpy as np
import pytest

from paper_2411_11833_amd import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

NONE = 2 ** 31 - 1


def _adam(n):
    from paper_2411_11833_amd.binding import CtAdam
    return CtAdam(1e-2, 0.9, 0.999, 1e-8, 1.0 / n)


def _state(gp, n, seed):
    X, M, V = gp.empty(n), gp.empty(n), gp.empty(n)
    gp.seed_uniform(seed, X, M, V, n)
    cost, mask = torch.zeros(n, device="cuda"), torch.zeros(n, dtype=torch.uint8, device="cuda")
    return X, M, V, cost, mask, torch.full((1,), NONE, dtype=torch.int32, device="cuda")


def _same(a, b):
    torch.cuda.synchronize()
    return all(torch.equal(u, v) for u, v in zip(a, b))


@pytest.mark.parametrize("K,n,split,iters", [(1, 1, 4, 3), (1, 129, 1, 130), (4, 131, 2, 65), (6, 45, 4, 64),
                                              (5, 33, 1, 2)])
def test_iterations_of_one_launch_equal_single_steps(K, n, split, iters):
    from paper_2411_11833_amd.planner import GpuProblem, grasp_frozen
    gp = GpuProblem(I.packing(0, 1, n_objects=K, n_obstacles=3))
    gp.set_split(split)
    fz = grasp_frozen(gp.prob)
    a, b = _state(gp, n, 5), _state(gp, n, 5)
    gp.optimize(*a[:3], n, 0, iters, _adam(n), frozen=fz, cost=a[3], mask=a[4], first_sat=a[5])
    for t in range(1, iters + 1):
        gp.step(*b[:3], n, t, _adam(n), frozen=fz, cost=b[3], mask=b[4], first_sat=b[5])
    assert _same(a, b)


def _loose(tau):
    """Only the position errors decide Eq. (3): the tolerance sets when the
    first of 333 particles satisfies it (by the FP64 oracle's loop: 0.57 at
    once, 0.54 after about 24 iterations, 0.425 after about 60)."""
    prob = I.packing(0, 1, n_objects=2, n_obstacles=2)
    prob.tolerances = I.Tolerances(kin_pos=tau, kin_rot=4.0, grasp=1.0, place=9.0, jlim=9.0, coll=99.0)
    return prob


@pytest.mark.parametrize("split", [1, 2, 4])
@pytest.mark.parametrize("tau", [0.57, 0.54, 0.425, 0.0])
def test_stop_inside_a_launch(tau, split):
    from paper_2411_11833_amd.planner import GpuProblem
    gp = GpuProblem(_loose(tau))
    gp.set_split(split)
    n = 333
    a, b = _state(gp, n, 11), _state(gp, n, 11)
    for t in (0, 75):   # launches of 64 and 11 iterations, then one after the stop
        gp.optimize(*a[:3], n, t, 75, _adam(n), cost=a[3], mask=a[4], first_sat=a[5], stop_at_first=True)
    for t in range(150):
        gp.optimize(*b[:3], n, t, 1, _adam(n), cost=b[3], mask=b[4], first_sat=b[5], stop_at_first=True)
    assert _same(a, b)
    f = int(a[5].item())
    assert f == NONE if tau == 0.0 else f < 75


def test_stop_on_two_streams_shares_no_state():
    """The copies a stop-at-first launch keeps belong to the handle: a call on
    another stream waits for the one before it."""
    from paper_2411_11833_amd.planner import GpuProblem
    gp = GpuProblem(_loose(0.54))
    n = 333
    want = _state(gp, n, 11)
    gp.optimize(*want[:3], n, 0, 40, _adam(n), cost=want[3], mask=want[4], first_sat=want[5], stop_at_first=True)
    got = [_state(gp, n, 11) for _ in range(4)]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    for i, s in enumerate(got):
        with torch.cuda.stream(streams[i % 2]):
            gp.optimize(*s[:3], n, 0, 40, _adam(n), cost=s[3], mask=s[4], first_sat=s[5], stop_at_first=True)
    for s in got:
        assert _same(s, want)


@pytest.mark.parametrize("stop", [False, True])
def test_optimize_inside_a_captured_graph(stop):
    from paper_2411_11833_amd.planner import GpuProblem
    gp = GpuProblem(_loose(0.54))
    n, it = 333, 40
    want, got = _state(gp, n, 11), _state(gp, n, 11)
    start = [x.clone() for x in got]
    gp.optimize(*want[:3], n, 0, it, _adam(n), cost=want[3], mask=want[4], first_sat=want[5], stop_at_first=stop)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        gp.optimize(*got[:3], n, 0, it, _adam(n), cost=got[3], mask=got[4], first_sat=got[5], stop_at_first=stop)
    for _ in range(3):
        for x, x0 in zip(got, start):
            x.copy_(x0)
        g.replay()
        assert _same(got, want)
        other = _state(gp, n, 12)   # eager work between the replays
        gp.optimize(*other[:3], n, 0, 5, _adam(n), first_sat=other[5], stop_at_first=stop)
        torch.cuda.synchronize()
    assert np.isfinite(float(got[3].sum()))
