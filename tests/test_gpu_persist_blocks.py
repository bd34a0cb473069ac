"""Persistent execution with one element per thread and with several (the largest tile against
the workgroup), past the line of resident execution: states and gradients bitwise those of
the two-pass launches."""
import numpy as np
import pytest

from paper_2104_02646_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

CASES = {"tets": lambda: [W.batch_body(7, lo=1800, hi=2400), W.tiny_cube(1)], "cloth": lambda: [W.cloth(10, n=21)]}


@pytest.mark.parametrize("tile", [64, 256])
@pytest.mark.parametrize("case", sorted(CASES))
def test_blocks(case, tile):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2104_02646_amd import gsim as gs
    bodies = [b.round_to(np.float32) for b in CASES[case]()]

    def gradient(mode, block):
        m = gs.Model(bodies, torch.float32, max_steps=7, ckpt_every=3, tile_elems=tile)
        m.set_exec(mode)
        m.set_launch(1, block, 1)
        assert not m.runs_resident(7) and not m.runs_resident(7, backward=True)
        p = m.params_from_bodies()
        x0, v0 = (gs.soa(np.concatenate([getattr(b, k) for b in bodies])) for k in ("x0", "v0"))
        xT, vT = m.rollout(p, x0, v0, 7)
        g = m.zero_grads([k for k in ("mu", "lam", "ktri", "mass")])
        xb, vb = m.rollout_backward(p, 7, xT - x0, vT, g)
        torch.cuda.synchronize()
        return [xT, vT, xb, vb, *g.values()]
    ref = gradient(gs.EXEC_PLAIN, 256)
    for block in (64, 128, 256, 512):  # below, at and above the tiles
        for a, b in zip(ref, gradient(gs.EXEC_PERSIST, block)):
            assert torch.equal(a, b), (case, tile, block)
