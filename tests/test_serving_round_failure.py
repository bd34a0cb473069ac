"""A serving round that fails is issued again: the rounds planned ahead are dropped with it,
so no query skips a step.  On the host, over recorded launches."""
import numpy as np
import pytest

import hosthip
from paper_2104_02646_amd import workloads as W


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return hosthip.build(str(tmp_path_factory.mktemp("host")))


def calls(hip, fail=None):
    """The kernel launches of two queries' rounds, each round's with the first query's input
    state (as a pool offset) before its last one, and the number of errors."""
    from paper_2104_02646_amd import gsim as gs, serve
    e = serve.Engine(pool_bytes=128 << 20, max_live=4, device="cpu", stream=hip.stream)
    for k in range(2):
        b = W.tiny_cube(k).round_to(np.float32)
        e.submit(serve.QueryBuffers(b.with_params(target=b.x0), 9, 4))
    hip.reset()
    if fail:
        hip.fail(*fail)
    errors, done = 0, []
    for _ in range(100):
        try:
            nl, nq = e.tick()
        except gs.GsimError:
            errors += 1
            continue
        done += e.poll()
        if nl == 0 and nq == 0:
            break
    assert len(done) == 2
    base = e.pool.data_ptr()
    return [int(w[2:]) - base if w.startswith("x=") else w for w in hip.names()
            if w.startswith("x=") or w in ("mixed", "loss", "contact_reduce")], errors


@pytest.mark.parametrize("fail", [("mixed", 1), ("mixed", 3), ("mixed", 11), ("loss", 1), ("loss", 2),
                                  ("contact_reduce", 2)])
def test_failed_round_is_repeated(lib, monkeypatch, fail):
    hip = hosthip.use(lib, monkeypatch)
    want, errors = calls(hip)
    assert errors == 0 and want.count("mixed") == 20  # 9 forward, loss, 9 adjoint, end
    got, errors = calls(hip, fail)
    assert errors == 1
    at = [i for i, w in enumerate(want) if w == fail[0]][fail[1] - 1]  # the call that fails
    start = max([i + 1 for i, w in enumerate(want[:at]) if w == "mixed"], default=0)  # of its round
    assert got == want[:at + 1] + want[start:]
