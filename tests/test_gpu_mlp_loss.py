"""The loss of a training step, summed by 256 of the 512 threads of the
workgroup that ends it: row counts around that width, against the mean squared
error in float64 of the same outputs."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("rows", [64, 192, 256, 320, 512, 1024])
def test_loss_of_a_step(rows, weighted):
    from paper_2411_11833_amd.seeds import GpuMlp
    m = GpuMlp(d_feat=20, d_noise=4, depth=2, d_out=21, max_rows=1024)
    rng = np.random.default_rng(rows)
    m.set_params(np.concatenate([np.concatenate([rng.normal(0, (2 / i) ** 0.5, i * o), rng.normal(0, 0.1, o)])
                                 for i, o in m.dims]).astype(np.float32))
    feats, T = torch.randn(2, 20, device="cuda"), torch.randn(rows, 21, device="cuda")
    W = torch.rand(rows, 21, device="cuda") + 0.5 if weighted else None
    which = torch.randint(0, 2, (rows,), dtype=torch.int32, device="cuda")
    Y = m.forward(feats, rows, 7, which, keep=False).double()
    want = ((Y - T.double()) ** 2 * (1.0 if W is None else W.double())).mean().item()
    loss = torch.full((1,), -1.0, device="cuda")
    m.imle_step(feats, which, T, 1, 7, loss=loss, weights=W)
    # 21 + rows / 256 + 8 roundings of positive sums, and as many of the squares
    assert abs(loss.item() - want) <= 1e-5 * want
