"""Tiles hold as many particles as deal a batch out evenly over the rounds of
512 tiles it takes; the lanes of a tile's empty columns share its tests.  The
results of a particle must not depend on it: batches on both sides of the
rule's lines against the same particles in a batch of full tiles, bit for
bit."""
import pytest

from paper_2411_11833_amd import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _run(prob, split, n, X):
    from paper_2411_11833_amd.binding import CtAdam
    from paper_2411_11833_amd.planner import GpuProblem
    gp = GpuProblem(prob)
    gp.set_split(split)
    Xd = gp.from_rows(X[:n])
    c0, T, m0 = gp.cost(Xd, n, terms=True)
    pairs = gp.penetrating_pairs(Xd, n)
    _, G = gp.cost_grad(Xd, n)
    M, V = torch.zeros_like(Xd), torch.zeros_like(Xd)
    c, m = torch.zeros(n, device="cuda"), torch.zeros(n, dtype=torch.uint8, device="cuda")
    gp.optimize(Xd, M, V, n, 0, 5, CtAdam(1e-2, 0.9, 0.999, 1e-8, 1.0), cost=c, mask=m)
    torch.cuda.synchronize()
    cols = [a[:, :n] for a in (T, G, Xd, M, V)]
    return [a.clone() for a in [c0, m0, pairs, c, m, *cols]]


@pytest.mark.parametrize("K,split,n", [(1, 1, 2), (1, 1, 16 * 512 + 1), (1, 1, 128 * 512 + 1), (1, 4, 511), (2, 4, 1025),
                                       (2, 2, 4096), (3, 4, 5), (3, 2, 7700), (4, 1, 515), (4, 4, 4097), (5, 2, 1537),
                                       (6, 4, 1), (6, 4, 1501), (6, 4, 2561)])
@pytest.mark.parametrize("self_collision", [0, 1])
def test_small_batches_equal_full_tiles(K, split, n, self_collision):
    prob = I.packing(K, 1, n_objects=K, n_obstacles=3)
    prob.skeleton.self_collision = self_collision
    tiles = 512 * (256 // (2 * K * split))
    full = -(-n // tiles) * tiles   # whole rounds of full tiles
    X = I.uniform_particles(prob, full, seed=5)
    small, large = _run(prob, split, n, X), _run(prob, split, full, X)
    for a, b in zip(small, large):
        assert torch.equal(a, b[..., :n])


@pytest.mark.parametrize("sizes", [[33, 1], [2048, 2100], [6000, 9000, 1]])
def test_small_batches_of_skeletons_equal_single_launches(sizes):
    """The many-skeleton kernel sizes its tiles over all of its skeletons, a
    single launch its own."""
    from paper_2411_11833_amd.binding import CtAdam
    from paper_2411_11833_amd.planner import GpuBatch
    probs = [I.packing(s, 1, n_objects=k, n_obstacles=2) for s, k in enumerate([1, 6, 3][:len(sizes)])]
    out = []
    for persistent in (True, False):
        b = GpuBatch(probs, sizes)
        b.set_tuning(1, 0, persistent)
        b.seed(4)
        b.optimize(0, 4, CtAdam(1e-2, 0.9, 0.999, 1e-8, 1.0))
        torch.cuda.synchronize()
        out.append([x.clone() for s in range(len(sizes)) for x in (b.X[s], b.M[s], b.V[s], b.cost[s], b.mask[s])])
    assert all(torch.equal(u, v) for u, v in zip(*out))
