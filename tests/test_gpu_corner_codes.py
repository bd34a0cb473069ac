"""Corner codes at the edges of what they hold: a fan whose hub has more corners than a code
counts in one tile (the tile ends early), tiles of the most elements and particles, and
meshes of single elements; four steps and their gradient against float64."""
import numpy as np
import pytest

from paper_2104_02646_amd import gsim as G
from paper_2104_02646_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def fan(n):
    """n tets around one axis: both axis particles are in every tet."""
    a = np.linspace(0, 2 * np.pi, n, endpoint=False)
    X = np.concatenate([[[0, 0, 0], [0, 1, 0]], np.stack([np.cos(a), 0.5 + 0 * a, np.sin(a)], 1)])
    i = np.arange(n)
    tets = np.stack([0 * i, 0 * i + 1, 2 + i, 2 + (i + 1) % n], 1).astype(np.int32)
    return X, tets


def loose(n):
    """n tets that share no particle."""
    X = np.concatenate([np.array([[0, 0, 0], [1, 0, 0], [0, 1, 0], [0, 0, 1.0]]) + [2.0 * k, 0, 0] for k in range(n)])
    return X, np.arange(4 * n, dtype=np.int32).reshape(-1, 4)


@pytest.mark.parametrize("mesh,n,tile", [("fan", 63, 0), ("fan", 64, 0), ("fan", 65, 0), ("fan", 200, 2048),
                                         ("loose", 1, 0), ("loose", 255, 512), ("loose", 256, 512), ("loose", 300, 2048)])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_corner_codes(mesh, n, tile, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    G.load()
    rng = np.random.default_rng(n)
    X, tets = fan(n) if mesh == "fan" else loose(n)
    b = W.Body(X=X, tets=tets, mu=rng.uniform(1e3, 2e3, n), lam=rng.uniform(1e3, 2e3, n), mass=rng.uniform(0.5, 1, len(X)),
               ground=False, dt=1e-3)
    b = b.round_to(np.float32)
    t = torch.float64 if dtype == "f64" else torch.float32
    m = G.Model([b], t, max_steps=4, ckpt_every=2, tile_elems=tile)
    p = m.params_from_bodies()
    x = (X + rng.normal(0, 1e-2, X.shape)).astype(np.float32)
    v = rng.normal(0, 1, X.shape).astype(np.float32)
    xT, vT = m.rollout(p, G.soa(x, t), G.soa(v, t), 4)
    w = rng.normal(size=X.shape).astype(np.float32)
    g = m.zero_grads(("mu", "lam", "mass"))
    xb, vb = m.rollout_backward(p, 4, G.soa(w, t), G.soa(0 * w, t), g)
    torch.cuda.synchronize()
    # the same four steps in float64 torch (compressible Neo-Hookean, semi-implicit Euler)
    f8 = lambda a: torch.as_tensor(np.asarray(a, np.float64))
    mu, lam, mass, x0, v0 = (f8(a).requires_grad_(True) for a in (b.mu, b.lam, b.mass, x, v))
    T4 = torch.as_tensor(tets.astype(np.int64))
    edges = lambda q: torch.stack([q[T4[:, k]] - q[T4[:, 0]] for k in (1, 2, 3)], 2)
    Dm = edges(f8(b.X))
    det = torch.linalg.det(Dm)
    inv, vol = torch.linalg.inv(Dm), det.abs() / 6
    q, u = x0, v0
    for _ in range(4):
        F = edges(q) @ inv
        Ic, J = (F * F).sum((1, 2)), torch.linalg.det(F)
        alpha = 1 + 0.75 * mu / lam
        cof = J[:, None, None] * torch.linalg.inv(F).transpose(1, 2)
        P = (mu * (1 - 1 / (Ic + 1)))[:, None, None] * F + (lam * (J - alpha))[:, None, None] * cof
        H = -vol[:, None, None] * P @ inv.transpose(1, 2)
        f = torch.zeros_like(q)
        for k in range(3):
            f = f.index_add(0, T4[:, k + 1], H[:, :, k]).index_add(0, T4[:, 0], -H[:, :, k])
        u = u + b.dt * (f / mass[:, None] + f8(b.gravity))
        q = q + b.dt * u
    (q * f8(w)).sum().backward()
    # float32: four steps of forces of up to 200 corners, each rounded to 2^-24 of the largest
    tol = 2e-5 if dtype == "f32" else 1e-11
    rel = lambda a, c: np.abs(a - c).max() / np.abs(c).max()
    assert rel(G.aos(xT), q.detach().numpy()) <= tol and rel(G.aos(vT), u.detach().numpy()) <= tol
    grads = {"mu": mu.grad, "lam": lam.grad, "mass": mass.grad}
    for k, ref in grads.items():
        assert rel(g[k].double().cpu().numpy().reshape(-1), ref.numpy()) <= 50 * tol, k
    assert rel(G.aos(xb), x0.grad.numpy()) <= 5 * tol and rel(G.aos(vb), v0.grad.numpy()) <= 5 * tol
