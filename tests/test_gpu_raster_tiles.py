"""Soft silhouette at the edges of its kernels' splits: images of 8 x 8 and of 4 x 4 pixel
tiles with ragged borders, chunks of 64 triangles with remainders, more chunks than one
lookup tests, meshes of a workgroup and of a wavefront per triangle; image and gradient
against the float64 oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def soup(nt, H, Wd, rng):
    """nt triangles of about 3 pixels, one per 20 square pixels around the image's centre
    (or over the whole image when they are few), in both orientations."""
    r = max((20.0 * nt) ** 0.5 / 2, 0.6 * max(H, Wd) / 2)
    uv = np.array([Wd / 2, H / 2]) + rng.uniform(-r, r, (nt, 1, 2)) + rng.uniform(-3, 3, (nt, 3, 2))
    X = np.concatenate([uv, np.ones((nt, 3, 1))], axis=2).reshape(-1, 3)
    return np.arange(3 * nt, dtype=np.int32).reshape(-1, 3), X.astype(np.float32).astype(np.float64)


@pytest.mark.parametrize("nt,H,Wd", [(1, 9, 13), (63, 60, 61), (65, 124, 124), (65, 129, 128), (1024, 40, 37),
                                     (1025, 40, 37), (513, 130, 131), (32833, 12, 13)])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_tiles_and_chunks(nt, H, Wd, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2104_02646_amd import gsim as gs
    gs.load()
    from oracle import raster as R
    dt = torch.float32 if dtype == "f32" else torch.float64
    rng = np.random.default_rng(nt)
    tris, X = soup(nt, H, Wd, rng)
    P, sigma = np.eye(3, 4), 0.7
    ibar = rng.normal(size=(H, Wd)).astype(np.float32).astype(np.float64)
    r = gs.Renderer(tris, len(X), H, Wd, dt)
    x = gs.soa(X, dt)
    img = r.forward(x, P, sigma)
    xb = r.backward(x, P, sigma, torch.as_tensor(ibar).to("cuda", dt))
    assert torch.equal(img, r.forward(x, P, sigma))
    Xo = torch.tensor(X, dtype=torch.float64, requires_grad=True)
    ref = R.silhouette(Xo, torch.as_tensor(tris, dtype=torch.long), torch.tensor(P), H, Wd, sigma)
    (ref * torch.tensor(ibar)).sum().backward()
    # float32: a pixel coordinate of up to 130 rounds by 8e-6, which moves x = d^2 / sigma by
    # up to 2 * 3.1 * 8e-6 / 0.7 = 7e-5 and the image by less; terms that rounding puts on
    # the other side of the cut-off move it by 1e-6 each; their share of a gradient is the same
    img_tol, g_tol = (2e-4, 2e-3) if dtype == "f32" else (1e-11, 1e-9)
    assert np.abs(img.double().cpu().numpy() - ref.detach().numpy()).max() <= img_tol
    want = Xo.grad.numpy()
    assert np.abs(gs.aos(xb) - want).max() <= g_tol * np.abs(want).max()
