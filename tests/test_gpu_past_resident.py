"""The two-pass, shared and persistent kernels on bodies of tets past the line of resident
execution (smaller ones run none of them), each test saying so first: the block of the
element passes, the overlapped backward, its paired layout and the execution modes, bitwise
against each other and against the FP64 oracle."""
import numpy as np
import pytest

from helpers import oracle_for, rel
from paper_2104_02646_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def gs():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2104_02646_amd import gsim
    gsim.load()
    return gsim


def bodies_of(n, lo, hi, dtype, seed=63000):
    out = [W.batch_body(seed + i, lo=lo, hi=hi) for i in range(n)]
    return [b.round_to(np.float32) for b in out] if dtype == torch.float32 else out


def gradient(gs, bodies, dtype, T, K, mode, overlap=True, tile=0, block=256, lanes=1, targets=None):
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        m = gs.Model(bodies, dtype, max_steps=T, ckpt_every=K, overlap=overlap, tile_elems=tile)
        m.set_exec(mode)
        m.set_launch(0, block, 1)
        m.set_lanes(lanes)
        for n in (1, T):
            assert not m.runs_resident(n) and not m.runs_resident(n, backward=True)
        p = m.params_from_bodies()
        x0, v0 = (gs.soa(np.concatenate([getattr(b, k) for b in bodies]), dtype) for k in ("x0", "v0"))
        tg = x0 + 0.01 if targets is None else gs.soa(np.concatenate(targets), dtype)
        xT, vT = m.rollout(p, x0, v0, T, stream=stream)
        loss, xb, vb = m.loss_mse(xT, tg, stream=stream)
        g = m.zero_grads(("mu", "lam", "mass", "contact"))
        xb0, vb0 = m.rollout_backward(p, T, xb, vb, g, stream=stream)
        stream.synchronize()
    out = {"x": xT, "v": vT, "loss": loss, "xb": xb0, "vb": vb0, **g}
    return {k: t.detach().cpu().numpy() for k, t in out.items()}


def same(a, b, what):
    for k in a:
        assert np.isfinite(a[k]).all() and np.array_equal(a[k], b[k]), (k, what)


def test_the_line(gs):
    """Bodies on both sides of it."""
    small, large = gs.Model([W.tiny_cube(0)], max_steps=9), gs.Model(bodies_of(1, 1800, 2000, torch.float32), max_steps=9)
    assert small.runs_resident(9) and small.runs_resident(9, backward=True) and not large.runs_resident(9)
    assert not gs.Model([W.tiny_cube(0)], torch.float64, max_steps=9).runs_resident(9)
    small.set_launch(1, 256, 2)
    assert not small.runs_resident(9)


@pytest.mark.parametrize("tile, blocks", [(64, (64, 256)), (128, (64, 128, 512)), (2048, (64, 192, 512))])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_block_does_not_change_a_bit(gs, dtype, tile, blocks):
    dt = torch.float32 if dtype == "f32" else torch.float64
    bodies = bodies_of(2, 1800, 2600, dt)
    for overlap in (False, True):
        ref = gradient(gs, bodies, dt, 12, 4, gs.EXEC_PLAIN, overlap, tile, blocks[0])
        for block in blocks[1:]:
            same(ref, gradient(gs, bodies, dt, 12, 4, gs.EXEC_PLAIN, overlap, tile, block), (overlap, block))


@pytest.mark.parametrize("T,K", [(40, 7), (12, 1), (9, 10), (30, 29)])
def test_overlap_equals_sequential(gs, T, K):
    bodies = bodies_of(1, 1800, 2600, torch.float32)
    ref = gradient(gs, bodies, torch.float32, T, K, gs.EXEC_PLAIN, overlap=False)
    for mode in (gs.EXEC_PLAIN, gs.EXEC_GRAPH, gs.EXEC_PERSIST):
        same(ref, gradient(gs, bodies, torch.float32, T, K, mode), mode)


@pytest.mark.parametrize("tile,block,lo,hi", [(32, 64, 2000, 5000), (128, 64, 13000, 16000)])  # one element per thread, and two
@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_paired_layout_equals_sequential(gs, dtype, tile, block, lo, hi):
    """At least 2048 element tiles: the shared element launch pairs a tile's two passes in
    one workgroup.  One lane and three, plain execution."""
    dt = torch.float32 if dtype == "f32" else torch.float64
    bodies = bodies_of(20, lo, hi, dt, 62000)
    assert len(gs.Plan(bodies, dt, tile).tiles()[0]) >= 2048
    ref = gradient(gs, bodies, dt, 9, 4, gs.EXEC_PLAIN, False, tile, block)
    for lanes in (1, 3):
        same(ref, gradient(gs, bodies, dt, 9, 4, gs.EXEC_PLAIN, True, tile, block, lanes), lanes)


def test_overlap_and_persistent_against_oracle(oracle_lib, gs):
    """One body of about 2000 tets, FP32, 60 steps, checkpoints every 10: positions within 1e-4
    and gradients within 1e-3 of the FP64 oracle."""
    body, = bodies_of(1, 1800, 2200, torch.float32)
    tgt = W.synthetic_target(body, 1).astype(np.float32).astype(np.float64)
    L, go, xs, _ = oracle_for(oracle_lib, body).loss_and_grad(body.params(), body.x0, body.v0, 60, tgt,
                                                               want=("mu", "lam", "mass"))
    for mode in (gs.EXEC_GRAPH, gs.EXEC_PERSIST):
        got = gradient(gs, [body], torch.float32, 60, 10, mode, targets=[tgt])
        errs = {k: rel(got[k].ravel(), np.ravel(go[k])) for k in ("mu", "lam", "mass", "contact")}
        errs["x"] = rel(got["x"].T, xs[-1])
        print(mode, {k: "%.2e" % v for k, v in errs.items()})
        assert errs.pop("x") < 1e-4 and abs(got["loss"][0] - L) < 1e-3 * L and all(v < 1e-3 for v in errs.values())
