"""Bodies with one particle in every element."""
import numpy as np

from paper_2104_02646_amd import workloads as W


def tet_fan(n):
    """n tets around one axis: both axis particles are in every tet."""
    rng = np.random.default_rng(n)
    a = np.linspace(0, 2 * np.pi, n, endpoint=False)
    X = np.concatenate([[[0, 0, 0], [0, 1, 0]], np.stack([np.cos(a), 0.5 + 0 * a, np.sin(a)], 1)])
    i = np.arange(n)
    tets = np.stack([0 * i, 0 * i + 1, 2 + i, 2 + (i + 1) % n], 1).astype(np.int32)
    return _moving(W.Body(X=X, tets=tets, mu=rng.uniform(1e3, 2e3, n), lam=rng.uniform(1e3, 2e3, n),
                          mass=rng.uniform(0.5, 1, len(X)), ground=False, dt=1e-4), rng)


def disc(n, air=False):
    """n triangles around one particle, hinges on their inner edges."""
    rng = np.random.default_rng(n)
    a = np.linspace(0, 2 * np.pi, n, endpoint=False)
    X = np.concatenate([[[0, 0.1, 0]], np.stack([np.cos(a), 0 * a, np.sin(a)], 1)])
    i = np.arange(n)
    tris = np.stack([0 * i, 1 + i, 1 + (i + 1) % n], 1).astype(np.int32)
    return _moving(W.Body(X=X, tris=tris, hinges=W.hinges_from_tris(tris), ktri=rng.uniform(1e3, 2e3, n),
                          mass=rng.uniform(0.5, 1, len(X)), kb=0.01, ground=False, dt=1e-4, air=air, kdrag=2.0 * air,
                          klift=2.0 * air), rng)


def _moving(b, rng):
    return b.with_params(x0=b.X + rng.normal(0, 1e-4, b.X.shape), v0=rng.normal(0, 0.1, b.X.shape)).round_to(np.float32)
