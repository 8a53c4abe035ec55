"""The many-skeleton kernel has one compiled tile per skeleton length: every
length, ragged sizes and a workgroup count that makes one workgroup run tiles
of different lengths in turn, bit for bit against one launch per skeleton of
the single-problem kernels (which are checked against the FP64 oracle)."""
import pytest

from paper_2411_11833_amd import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("self_collision", [False, True])
@pytest.mark.parametrize("split", [1, 2, 4])
def test_every_length_in_one_batch(split, self_collision):
    from paper_2411_11833_amd.binding import CtAdam
    from paper_2411_11833_amd.planner import GpuBatch
    lengths, sizes = [3, 1, 6, 2, 5, 4, 1], [61, 129, 45, 65, 1, 33, 7]
    probs = [I.packing(s, 1, n_objects=k, n_obstacles=s % 4) for s, k in enumerate(lengths)]
    for p in probs:
        p.skeleton.self_collision = int(self_collision)
    out = []
    for workgroups, persistent in ((3, True), (0, False)):
        b = GpuBatch(probs, sizes)
        b.set_tuning(split, workgroups, persistent)
        b.seed(4)
        for t0, iters in ((0, 3), (3, 66)):
            b.optimize(t0, iters, CtAdam(1e-2, 0.9, 0.999, 1e-8, 1.0))
        torch.cuda.synchronize()
        out.append([x.clone() for s in range(len(sizes))
                    for x in (b.X[s], b.M[s], b.V[s], b.cost[s], b.mask[s])] + [b.first_sat.clone()])
        b.close()
    assert all(torch.equal(u, v) for u, v in zip(*out))
