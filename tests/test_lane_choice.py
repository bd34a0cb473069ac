"""Choosing launch lanes: what was captured for the model's own choice is captured again, and a
choice that fails changes nothing.  On the host, over recorded HIP calls."""
import pytest

import hosthip
from paper_2104_02646_amd import workloads as W


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return hosthip.build(str(tmp_path_factory.mktemp("host")))


def test_graphs_follow_the_choice(lib, monkeypatch):
    """Two lanes chosen for a model that has two, but runs forward sequences on one while
    nobody has chosen (262144 to 458752 elements)."""
    from paper_2104_02646_amd import gsim as gs
    hip = hosthip.use(lib, monkeypatch)
    body = W.batch_body(7, lo=14000, hi=15000)
    m, p, x, v = hip.model([body] * (300000 // body.ne), max_steps=3, ckpt_every=3)
    m.set_exec(gs.EXEC_GRAPH)
    m.step(p, x, v, 3, stream=hip.stream)
    hip.reset()
    m.step(p, x, v, 3, stream=hip.stream)
    assert hip.count()["capture"] == 0 and m.get_lanes() == 2
    m.set_lanes(2)
    hip.reset()
    m.step(p, x, v, 3, stream=hip.stream)
    n = hip.count()
    assert n["capture"] == 1 and n["elem_fwd"] == 6 and n["wait_event"] == 2, n
    hip.reset()
    m.set_lanes(2)  # chosen already: nothing to do
    assert hip.names() == []


@pytest.mark.parametrize("what,nth", [("stream", 1), ("event", 1), ("event", 2), ("device_sync", 1)])
def test_failed_choice_changes_nothing(lib, monkeypatch, what, nth):
    from paper_2104_02646_amd import gsim as gs
    hip = hosthip.use(lib, monkeypatch)
    m, p, x, v = hip.model([W.batch_body(k, lo=3000, hi=4000) for k in (1, 2)], max_steps=2, ckpt_every=2)
    hip.reset()
    hip.fail(what, nth)
    with pytest.raises(gs.GsimError):
        m.set_lanes(2)
    hip.reset()
    m.step(p, x, v, 2)
    n = hip.count()
    assert n["elem_fwd"] == 2 and n["wait_event"] == 0, n  # one lane, as before
    m.set_lanes(2)
    hip.reset()
    m.step(p, x, v, 2)
    n = hip.count()
    assert n["elem_fwd"] == 4 and n["wait_event"] == 2, n


def test_tuner_times_no_lanes_twice(lib, monkeypatch):
    """Each of the tuner's lane candidates runs a number of lanes of its own."""
    from paper_2104_02646_amd import autotune
    hip = hosthip.use(lib, monkeypatch)
    m, p, x, v = hip.model([W.batch_body(k, lo=3000, hi=4000) for k in range(4)], max_steps=1)
    ran = []
    for lanes in autotune.LANE_CANDIDATES:
        m.set_lanes(lanes)
        hip.reset()
        m.step(p, x, v, 1)
        ran.append(hip.count()["elem_fwd"])
    assert ran == sorted(set(ran)) and ran[0] == 1, ran
