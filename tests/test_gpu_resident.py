"""Resident execution (small tet bodies stay on one compute unit for a call's whole run of
steps) against the two-pass launches, which run whenever a kernel is timed: every output
bitwise equal.  Bodies at the edges of the tets-per-thread variants and of the workgroup,
pinned and unattached particles, several bodies of different size, every checkpoint
pattern, held and per-step actuation with gradients, every block of the particle passes,
graph replay, aliased step states; and a body past the line, which keeps its launches."""
import numpy as np
import pytest

from paper_2104_02646_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def block(n_tets, seed=0, dims=None):
    """A box of Kuhn tets cut down to n_tets (some particles may carry none), on the ground."""
    dims = dims or next(d for d in ((3, 3, 3), (4, 4, 3), (6, 4, 4), (8, 6, 4), (10, 6, 5)) if 6 * np.prod(d) >= n_tets)
    X, tets = W.box_tets(*dims, 0.05)
    rng = np.random.default_rng(seed)
    X[:, 1] += 0.01
    pinned = (rng.random(len(X)) < 0.05).astype(np.uint8)
    b = W.Body(X=X, tets=tets[:n_tets], pinned=pinned, mu=rng.uniform(1e4, 1e5, n_tets), lam=rng.uniform(1e4, 1e5, n_tets),
               mass=rng.uniform(0.5, 1.5, len(X)), ke=1e4, kd=2.0, kf=100.0, muf=0.5, ground=True, dt=1 / 600,
               x0=X.copy(), v0=np.tile([1.0, -1.0, 0.0], (len(X), 1)))
    return b.round_to(np.float32)


def calls(bodies, T, K, timed, tile=0, pblock=256, act=None, graph=False, repeat=1):
    from paper_2104_02646_amd import gsim as gs
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        m = gs.Model(bodies, torch.float32, max_steps=T, ckpt_every=K, tile_elems=tile)
        m.set_launch(1, pblock, 1)
        if timed:
            m.set_timing()
        elif graph:
            m.set_exec(gs.EXEC_GRAPH)
        p = m.params_from_bodies()
        x0, v0 = (gs.soa(np.concatenate([getattr(b, k) for b in bodies])) for k in ("x0", "v0"))
        which, steps = ("mu", "lam", "mass", "contact"), None
        if act:
            rng = np.random.default_rng(4)
            shape = (T, m.ne) if act == "rows" else (m.ne,)
            p["act"] = torch.as_tensor(rng.normal(0, 0.05, shape), dtype=torch.float32, device="cuda")
            which, steps = which + ("act",), T if act == "rows" else None
        for _ in range(repeat):
            xT, vT = m.rollout(p, x0, v0, T)
            loss, xb, vb = m.loss_mse(xT, x0 + 0.01)
            g = {k: t + 0.5 for k, t in m.zero_grads(which, steps).items()}
            x0b, v0b = m.rollout_backward(p, T, xb, vb, g)
            xs, vs = x0.clone(), v0.clone()
            m.step(p, xs, vs, T, out=(xs, vs))
            x1, v1 = m.rollout(p, x0, v0, T, checkpoint=False)
            q = {k: v[0].contiguous() if k == "act" and act == "rows" else v for k, v in p.items()}
            g1 = {k: torch.zeros_like(t[0] if k == "act" and steps else t) for k, t in g.items()}
            xbm, vbm = m.step_backward(q, x0, v0, xb, vb, g1)
            torch.cuda.synchronize()
        flags = m.check()
    out = {"xT": xT, "vT": vT, "loss": loss, "x0b": x0b, "v0b": v0b, "xs": xs, "vs": vs, "x1": x1, "v1": v1,
           "xbm": xbm, "vbm": vbm, **g, **{"one_" + k: t for k, t in g1.items()}}
    return {k: t.cpu().numpy() for k, t in out.items()}, flags


def same(a, b):
    assert all(np.isfinite(t).all() for t in a[0].values())
    for k in a[0]:
        assert np.array_equal(a[0][k], b[0][k]), k
    assert np.array_equal(a[1], b[1])


@pytest.mark.parametrize("n_tets", [1, 6, 255, 256, 257, 512, 513, 1024, 1025, 1500])
def test_tets_per_thread_edges(n_tets):
    bodies = [block(n_tets, n_tets)]
    same(calls(bodies, 13, 5, True), calls(bodies, 13, 5, False))


@pytest.mark.parametrize("tile", [32, 100, 2048])
@pytest.mark.parametrize("T, K", [(1, 1), (6, 1), (7, 7), (12, 5)])
def test_tiles_and_checkpoints(tile, T, K):
    bodies = [block(300, 3), block(150, 4), block(1100, 5)]
    same(calls(bodies, T, K, True, tile=tile), calls(bodies, T, K, False, tile=tile))


@pytest.mark.parametrize("pblock", [64, 128, 512])
@pytest.mark.parametrize("act", ["held", "rows"])
def test_actuation_and_contact_tree(pblock, act):
    bodies = [W.tiny_cube(2).round_to(np.float32), W.gear().round_to(np.float32)]
    same(calls(bodies, 9, 4, True, pblock=pblock, act=act), calls(bodies, 9, 4, False, pblock=pblock, act=act))


def test_graph_replays():
    bodies = [W.walker().round_to(np.float32), W.tiny_cube(5).round_to(np.float32)]
    same(calls(bodies, 20, 6, True), calls(bodies, 20, 6, False, graph=True, repeat=4))


def test_past_the_line():
    bodies = [block(60, 6), block(1800, 7)]  # one body past it: the whole model keeps its launches
    same(calls(bodies, 6, 3, True), calls(bodies, 6, 3, False))
