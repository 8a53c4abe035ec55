"""The one-launch inference reads its weights from fragment-major copies and
the seeds leave through 64 x 32 tiles: output widths and row counts at the
edges of both, against the layer-by-layer forward pass (same operations in
the same order, so bit for bit) and the affine map of its outputs."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _mlp(d_out, depth, d_feat, d_noise, rows):
    from paper_2411_11833_amd.seeds import GpuMlp
    m = GpuMlp(d_feat=d_feat, d_noise=d_noise, depth=depth, d_out=d_out, max_rows=rows)
    rng = np.random.default_rng(d_out + depth)
    m.set_params(np.concatenate([np.concatenate([rng.normal(0, (2 / i) ** 0.5, i * o), rng.normal(0, 0.1, o)])
                                 for i, o in m.dims]).astype(np.float32))
    return m


@pytest.mark.parametrize("d_out,depth,d_feat,d_noise", [(1, 1, 0, 32), (16, 2, 28, 4), (33, 3, 120, 32),
                                                        (96, 8, 4, 8), (97, 1, 480, 32), (128, 3, 64, 0)])
@pytest.mark.parametrize("rows", [8192 + 64, 16384 + 64, 32768 + 64])
def test_one_launch_inference_equals_layers(d_out, depth, d_feat, d_noise, rows):
    m = _mlp(d_out, depth, d_feat, d_noise, rows)
    feats = torch.randn(3, max(d_feat, 1), device="cuda")
    which = torch.randint(0, 3, (rows,), dtype=torch.int32, device="cuda")
    draw = torch.randint(0, 9, (rows,), dtype=torch.int32, device="cuda")
    fused = m.forward(feats, rows, 11, which, draw, keep=False)
    # batches below the one-launch range take the per-layer kernels; a row's
    # noise depends on its index, so compare the first rows
    part = m.forward(feats, 4096, 11, which, draw, keep=False)
    assert torch.equal(fused[:4096], part)
    m.t = 0
    dY = torch.randn(rows, d_out, device="cuda")
    m.forward(feats, rows, 11, which, draw, keep=True)
    m.backward(dY, rows)
    m.adam(1e-2)   # refreshes every copy of the weights
    assert torch.equal(m.forward(feats, rows, 11, which, draw, keep=False)[:4096],
                       m.forward(feats, 4096, 11, which, draw, keep=False))


@pytest.mark.parametrize("d_out,n", [(1, 1), (31, 63), (32, 64), (33, 65), (84, 130), (128, 8200)])
def test_seed_tiles(d_out, n):
    rows = (n + 63) // 64 * 64
    m = _mlp(d_out, 2, 20, 32, rows)
    feats = torch.randn(1, 20, device="cuda")
    Y = m.forward(feats, n, 5, keep=False).double().cpu()
    mean, std = torch.randn(d_out, device="cuda"), torch.rand(d_out, device="cuda") + 0.5
    wrap = (torch.arange(d_out, device="cuda") % 3 == 0).to(torch.uint8)
    lo, hi = torch.full((d_out,), -2.0, device="cuda"), torch.full((d_out,), 2.5, device="cuda")
    X, M, V = (torch.full((d_out, rows + 64), 7.0, device="cuda") for _ in range(3))
    m.sample(feats, 5, mean, std, lo, hi, wrap, X, M, V, n)
    torch.cuda.synchronize()
    for a in (X, M, V):
        assert torch.all(a[:, n:] == 7)
    assert torch.all(M[:, :n] == 0) and torch.all(V[:, :n] == 0)
    mu, sd, w = mean.double().cpu(), std.double().cpu(), wrap.bool().cpu()
    x = Y * sd + mu
    # a few roundings of the largest magnitude met: |y std| + |mean| and, wrapped, multiples of 2 pi
    tol = (Y.abs() * sd + mu.abs() + 7) * 2.0 ** -21
    turns = torch.floor((x + np.pi) / (2 * np.pi))
    near = (torch.remainder(x + np.pi, 2 * np.pi) - np.pi).abs() > np.pi - 1e-4
    want = torch.where(w, x - 2 * np.pi * turns, x).clamp(-2.0, 2.5)
    err = (X[:, :n].double().cpu().T - want).abs()
    assert torch.all((err <= tol) | (near & w))
