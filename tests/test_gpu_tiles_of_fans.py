"""Particles of more corners in a tile than a code's rank counts: three steps and their
gradient in tiles of 32 elements, where no particle has more, and in larger ones.  Only
the order of the sums differs: n terms of 2^-53 (2^-24) each, over three steps."""
import numpy as np
import pytest

from fans import disc, tet_fan

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

BODIES = {"fan 33": lambda: tet_fan(33), "fan 65": lambda: tet_fan(65), "fan 300": lambda: tet_fan(300),
          "fan 3000": lambda: tet_fan(3000), "disc 33": lambda: disc(33), "disc 500": lambda: disc(500),
          "disc 500 air": lambda: disc(500, True)}


def gradient(gs, body, dtype, tile):
    m = gs.Model([body], dtype, max_steps=3, ckpt_every=2, tile_elems=tile)
    p = m.params_from_bodies()
    xT, vT = m.rollout(p, gs.soa(body.x0, dtype), gs.soa(body.v0, dtype), 3)
    w = np.random.default_rng(1).normal(size=body.X.shape)
    g = m.zero_grads()
    xb, vb = m.rollout_backward(p, 3, gs.soa(w, dtype), gs.soa(0 * w, dtype), g)
    torch.cuda.synchronize()
    return {k: t.double().cpu().numpy() for k, t in {"x": xT, "v": vT, "xb": xb, "vb": vb, **g}.items()}


@pytest.mark.parametrize("name", list(BODIES))
@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_further_entries(name, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2104_02646_amd import gsim as gs
    gs.load()
    body = BODIES[name]()
    dt = torch.float32 if dtype == "f32" else torch.float64
    n = body.ne + body.nt + body.nh
    tol = 8 * n * 2.0 ** (-24 if dtype == "f32" else -53)
    ref = gradient(gs, body, dt, 32)
    for tile in (0, 512, 2048):
        got = gradient(gs, body, dt, tile)
        for k, a in ref.items():
            assert np.abs(got[k] - a).max() <= tol * max(np.abs(a).max(), 1e-30), (k, tile)
