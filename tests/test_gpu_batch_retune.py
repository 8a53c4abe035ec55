"""ct_batch_set_tuning and ct_batch_autotune replace the tables that the
batch's launches read.  A launch still running on a stream that the legacy
stream does not wait for keeps its own: bit for bit against the same calls with
a wait for the device before every change."""
import pytest

from paper_2411_11833_amd import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _run(wait, tune):
    from paper_2411_11833_amd.binding import CtAdam
    from paper_2411_11833_amd.planner import GpuBatch
    sizes = [1500, 700, 2000]
    b = GpuBatch([I.packing(s, 1, n_objects=k, n_obstacles=2) for s, k in enumerate((4, 2, 6))], sizes)
    b.set_tuning(1, 24)   # many items for each workgroup: most are taken after the change below
    b.seed(4)
    adam = CtAdam(1e-2, 0.9, 0.999, 1e-8, 1.0)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    t = 0
    with torch.cuda.stream(side):
        for split in (2, 1, 4):
            b.optimize(t, 64, adam)
            t += 64
            if wait:
                torch.cuda.synchronize()
            if tune:
                b.autotune()
            b.set_tuning(split, 24)
        b.optimize(t, 2, adam)
    torch.cuda.synchronize()
    out = [x.clone() for s in range(len(sizes)) for x in (b.X[s], b.M[s], b.V[s], b.cost[s], b.mask[s])]
    b.close()
    return out


@pytest.mark.parametrize("tune", [False, True])
def test_tuning_changed_while_a_launch_runs(tune):
    assert all(torch.equal(u, v) for u, v in zip(_run(False, tune), _run(True, tune)))
