"""ct_step_mask on more particles than one launch has threads for at four a
particle (2^32): 2^30 of one step, whose terms take 48 GB."""
import pytest

from paper_2411_11833_amd import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_more_particles_than_a_launch_holds():
    from paper_2411_11833_amd.planner import GpuProblem
    n = (1 << 30) + 1
    ld = (n + 63) // 64 * 64
    if torch.cuda.mem_get_info()[0] < 80 << 30:
        pytest.skip("needs 60 GB of device memory")
    gp = GpuProblem(I.single_pick_place(0, 0))
    T = torch.zeros((gp.n_terms, ld), device="cuda")
    off = torch.tensor([0, (1 << 28) - 1, 1 << 28, (1 << 30) - 1, n - 1], device="cuda")
    T[3, off] = 100.0      # one term beyond its tolerance
    T[7, off[1]] = float("nan")
    mask, count = gp.step_mask(T, n)
    del T
    assert count[off].tolist() == [10, 9, 10, 10, 10] and not mask[0, off].any()
    assert int((count == 11).sum()) == int((mask[0, :n] == 1).sum()) == n - 5
    del mask, count
    torch.cuda.empty_cache()
