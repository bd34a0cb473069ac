"""Launch lanes that nobody chose: a model runs on one lane, on two, or on one for its
forward sequences alone, by its count of elements.  Results are bitwise those of
lanes set explicitly, on each side of both thresholds and with lift/drag bodies mixed in."""
import numpy as np
import pytest
import torch

from paper_2104_02646_amd import workloads as W

pytestmark = pytest.mark.gpu


def run(gs, m, bodies, stream, T=6):
    with torch.cuda.stream(stream):
        p = m.params_from_bodies()
        x0, v0 = (gs.soa(np.concatenate([getattr(b, k) for b in bodies]), dtype=torch.float32) for k in ("x0", "v0"))
        tg = gs.soa(np.concatenate([W.synthetic_target(b, 7 + i) for i, b in enumerate(bodies)]), dtype=torch.float32)
        xT, vT = m.rollout(p, x0, v0, T, stream=stream)
        loss, xb, vb = m.loss_mse(xT, tg, stream=stream)
        g = m.zero_grads(("mu", "lam", "ktri", "mass", "contact"))
        xb0, vb0 = m.rollout_backward(p, T, xb, vb, g, stream=stream)
        stream.synchronize()
    out = {"x": xT, "v": vT, "loss": loss, "xb": xb0, "vb": vb0, **g}
    return {k: v.detach().cpu().numpy() for k, v in out.items()}


@pytest.mark.parametrize("case", ["small", "mixed air", "forward", "many"])
def test_default_lanes_bitwise(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2104_02646_amd import gsim as gs
    gs.load()
    n, lo, hi = {"small": (3, 2800, 4000), "mixed air": (2, 2800, 4000), "forward": (24, 12000, 15000),
                 "many": (40, 12000, 15000)}[case]
    bodies = [W.batch_body(5000 + i, lo=lo, hi=hi).round_to(np.float32) for i in range(n)]
    if case == "mixed air":
        bodies += [W.control_cloth(31).round_to(np.float32), W.control_cloth(32).round_to(np.float32)]
    elements = sum(b.ne for b in bodies)  # between the thresholds of gradients and of rollouts, and above both
    assert case not in ("forward", "many") or (1 << 18 < elements < 7 << 16) == (case == "forward")
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        m = gs.Model(bodies, torch.float32, max_steps=6, ckpt_every=3)
    assert m.get_lanes() == 2
    ref = run(gs, m, bodies, stream)
    for lanes in (1, 2):
        m.set_lanes(lanes)
        assert m.get_lanes() == lanes
        got = run(gs, m, bodies, stream)
        for k in ref:
            assert np.array_equal(ref[k], got[k]), (k, lanes)
