"""Rounds planned ahead: a query's answer does not depend on how many rounds one table
upload holds (the engine's max_live bounds it: one round when every slot is taken) nor on
plans dropped because queries arrived between ticks."""
import numpy as np
import pytest

from paper_2104_02646_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("max_live,gap", [(3, 1), (3, 5), (64, 1), (64, 7), (64, 8)])
def test_answers_do_not_depend_on_planned_rounds(max_live, gap):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2104_02646_amd import serve as sv
    sv.gsim.load()
    eng = sv.Engine(pool_bytes=256 << 20, max_live=max_live)
    qbs = []
    for i, (T, K) in enumerate([(9, 4), (17, 17), (24, 5), (1, 1)]):
        b = W.batch_body(800 + i, lo=300, hi=900) if i % 2 else W.cloth(80 + i, n=9, size=0.5)
        b.target = W.synthetic_target(b, i)
        qbs.append(sv.QueryBuffers(b, T, K))
    n = 0
    for qb in qbs:  # one at a time, between them ticks that leave a plan partly used
        eng.submit(qb)
        for _ in range(gap):
            eng.tick()
            n += len(eng.poll())
    n += len(eng.run_until_idle())
    assert n == len(qbs) and eng.stats()["completed"] == len(qbs)
    for qb in qbs:
        loss, g = sv.solve_alone(qb)
        assert np.float32(loss) == np.float32(qb.loss)
        for k, v in (("mass", qb.out["mass"]), ("mu", qb.out["mu"]), ("lam", qb.out["lam"]), ("ktri", qb.out["k_tri"]),
                     ("contact", qb.out["contact"])):
            if v.size and k in g and g[k].size == v.size:
                assert np.array_equal(g[k], v), k
