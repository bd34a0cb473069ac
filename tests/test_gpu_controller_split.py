"""The controller's two layouts (eight wavefronts per 64 elements of a small layer, one per
64 of a large one) at the edges of their element groups, step batches and table chunks,
against float64."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n,N,T,t0", [(1, 1, 1, 0), (63, 3, 7, 5), (64, 16, 8, 0), (65, 8, 9, 1), (200, 8, 64, 0), (130, 5, 65, 0),
                                      (70, 8, 128, 3), (70, 2, 129, 0), (65535, 4, 11, 0), (65536, 4, 11, 0),
                                      (65601, 16, 130, 2)])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_layouts(n, N, T, t0, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2104_02646_amd import gsim as gs
    gs.load()
    dt = torch.float32 if dtype == "f32" else torch.float64
    rng = np.random.default_rng(n + T)
    W, g, gW0 = (rng.normal(size=s).astype(np.float32).astype(np.float64) for s in ((N, n), (T, n), (N, n)))
    omega, step, scale = 3.0, 1.0 / 64, 0.5
    dev = lambda a: torch.as_tensor(a).to("cuda", dt)
    act = gs.controller_forward(dev(W), omega, step, T, scale=scale, t0=t0)
    gW = gs.controller_backward(dev(W), dev(g), omega, step, scale=scale, t0=t0, W_grad=dev(gW0))
    tau = omega * step * (t0 + np.arange(T))
    S = np.sin(tau[:, None] + 2 * math.pi * np.arange(N) / N)  # [T, N]
    y = np.tanh(S @ W)
    want = gW0 + S.T @ (g * scale * (1 - y * y))
    # float32: A and B carry N roundings of terms |W|, z two more, tanh and its use a few:
    # 2^-23 (N + 8) max |W| sqrt(2) < 2e-5 for the layer; a weight gradient adds T + N terms of |g|
    eps = 2.0 ** -23 if dtype == "f32" else 2.0 ** -50
    wm = np.abs(W).max()
    layer = eps * (N + 8) * 1.5 * wm * N
    assert np.abs(act.double().cpu().numpy() - scale * y).max() <= scale * layer + eps
    got = gW.double().cpu().numpy()
    bound = np.abs(g).sum(0).max() * scale * (2 * layer + eps * (T + 8)) + eps * (1 + np.abs(gW0).max())
    assert np.abs(got - want).max() <= bound
