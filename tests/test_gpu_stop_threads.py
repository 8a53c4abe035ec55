"""Stop at the first satisfying particle on one handle from host threads that
take turns, each on hipStreamPerThread: one stream handle, but another stream
in every thread.  The copies that the launches keep belong to the handle, so a
call waits for the one before it."""
import threading

import pytest

from paper_2411_11833_amd import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

N = 333
PER_THREAD = 2   # hipStreamPerThread


def _state(gp, seed):
    X, M, V = gp.empty(N), gp.empty(N), gp.empty(N)
    gp.seed_uniform(seed, X, M, V, N)
    cost, mask = torch.zeros(N, device="cuda"), torch.zeros(N, dtype=torch.uint8, device="cuda")
    return X, M, V, cost, mask, torch.full((1,), 2 ** 31 - 1, dtype=torch.int32, device="cuda")


def test_calls_from_threads_wait_for_each_other():
    from paper_2411_11833_amd import binding as B
    from paper_2411_11833_amd.planner import GpuProblem
    prob = I.packing(0, 1, n_objects=2, n_obstacles=2)
    # satisfied after about 24 iterations: inside the launch, which is rolled back
    prob.tolerances = I.Tolerances(kin_pos=0.54, kin_rot=4.0, grasp=1.0, place=9.0, jlim=9.0, coll=99.0)
    gp = GpuProblem(prob)
    seeds = (11, 12, 13, 11)
    adam = B.CtAdam(1e-2, 0.9, 0.999, 1e-8, 1.0 / N)

    def solve(s, stream):
        B.ct_optimize(gp.handle, *(x.data_ptr() for x in s[:3]), N, s[0].shape[1], 0, 60, adam, None,
                      s[3].data_ptr(), s[4].data_ptr(), s[5].data_ptr(), 1, stream)

    want, got = [_state(gp, x) for x in seeds], [_state(gp, x) for x in seeds]
    torch.cuda.synchronize()
    for s in want:
        solve(s, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
    assert 0 < int(want[0][5].item()) < 59
    # one call after another, without a wait for the device; the threads stay,
    # as their streams go with them, whatever still runs there
    over, threads = threading.Event(), []
    for s in got:
        called = threading.Event()

        def work(s=s, called=called):
            try:
                solve(s, PER_THREAD)
            finally:
                called.set()
            over.wait()

        threads.append(threading.Thread(target=work))
        threads[-1].start()
        called.wait()
    torch.cuda.synchronize()
    over.set()
    for t in threads:
        t.join()
    for a, b in zip(got, want):
        assert all(torch.equal(u, v) for u, v in zip(a, b))
