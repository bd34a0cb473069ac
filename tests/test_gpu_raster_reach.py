"""A triangle reaches the pixels of its bounding box widened by the cut-off distance and no
others, in both tile layouts: a corner that projects to infinity leaves every pixel outside
that box as it is without the triangle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("first", [0, 1, 2])
@pytest.mark.parametrize("H,Wd", [(41, 42), (160, 161)])  # 4 x 4 and 8 x 8 tiles
@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_infinite_corner(dtype, H, Wd, first):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2104_02646_amd import gsim as gs
    gs.load()
    dt = torch.float32 if dtype == "f32" else torch.float64
    far = 3e38 if dtype == "f32" else 1e308
    z = 1e-3
    # a visible triangle, and one whose third corner has u = infinity and a finite v
    X = np.array([[9.0, 8.0, 1], [19.0, 11.0, 1], [14.0, 24.0, 1], [20.3, 9.0, 1], [20.6, 12.0, 1], [far, 10 * z, z]])
    T = np.array([[0, 1, 2], np.roll([3, 4, 5], first)], np.int32)
    P, sigma = np.eye(3, 4), 0.5
    x = torch.as_tensor(X.T.copy()).to("cuda", dt)
    img = gs.Renderer(T, 6, H, Wd, dt).forward(x, P, sigma).cpu().numpy()
    alone = gs.Renderer(T[:1], 6, H, Wd, dt).forward(x, P, sigma).cpu().numpy()
    r = np.sqrt(13.815510557964274 * sigma)
    c, row = np.meshgrid(np.arange(Wd) + 0.5, np.arange(H) + 0.5)
    out = (c < 20.3 - r) | (row < 9 - r) | (row > 12 + r)
    assert out.any(axis=1).all() and alone[out].max() > 0.9
    assert np.array_equal(img[out], alone[out])
