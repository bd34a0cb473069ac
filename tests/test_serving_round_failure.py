"""A serving round that fails is issued again: the rounds planned ahead are dropped with it,
so no query skips a step.  On the host, over recorded launches."""
import numpy as np
import pytest

import hosthip
from paper_2104_02646_amd import workloads as W


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return hosthip.build(str(tmp_path_factory.mktemp("host")))


def rounds(hip, fail=None):
    """The first query's input state of each round's launch (as a pool offset), and errors."""
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
    base = e.pool.data_ptr()
    assert len(done) == 2
    return [int(w[2:]) - base for w in hip.names() if w.startswith("x=")], errors


@pytest.mark.parametrize("fail", [("mixed", 1), ("mixed", 4), ("loss", 1), ("contact_reduce", 1)])
def test_failed_round_is_repeated(lib, monkeypatch, fail):
    hip = hosthip.use(lib, monkeypatch)
    want, errors = rounds(hip)
    assert errors == 0 and len(want) == 20
    got, errors = rounds(hip, fail)
    assert errors == 1
    if fail[0] == "mixed":  # the failed launch itself is among the calls
        at = fail[1] - 1
        assert got == want[:at + 1] + want[at:]
    else:  # it failed before the round's launch
        assert got == want
