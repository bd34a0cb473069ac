"""The launch-shape tuner and models whose calls run resident: a particle shape that wins among
the timed two-pass launches, or that the cache holds for the size, is not given to them.  On
the host, over recorded launches."""
import json

import pytest
import torch

import hosthip
from paper_2104_02646_amd import workloads as W


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return hosthip.build(str(tmp_path_factory.mktemp("host")))


@pytest.mark.parametrize("cached", [False, True])
def test_tuner_keeps_resident_models(lib, monkeypatch, tmp_path, cached):
    from paper_2104_02646_amd import autotune
    hip = hosthip.use(lib, monkeypatch)

    class Card:
        gcnArchName = "gfx950"
    monkeypatch.setattr(torch.cuda, "get_device_properties", lambda d: Card)
    cache = tmp_path / "tune.json"
    monkeypatch.setenv("GSIM_AUTOTUNE_CACHE", str(cache))
    # two particles per thread win among the launches
    monkeypatch.setattr(autotune, "_time_passes", lambda m, *a: dict.fromkeys(
        ("element_fwd", "particle_fwd", "element_adj", "particle_adj"), 1.0 / m.get_launch(1)[1]))

    def tuned(bodies):
        m, p, x, v = hip.model(bodies, max_steps=16, ckpt_every=5)
        if cached:
            with open(cache, "w") as f:
                json.dump({autotune.bucket_key(m, 1): {"shape": [256, 2]}}, f)
        before = m.runs_resident(16), m.runs_resident(16, backward=True)
        autotune.tune(m, p, x, v)
        return before, (m.runs_resident(16), m.runs_resident(16, backward=True)), m.get_launch(1)
    assert tuned([W.tiny_cube(0)]) == ((True, True), (True, True), (256, 1))
    large = [W.batch_body(5, lo=3000, hi=4000)]  # too large to be resident: tuned as before
    assert tuned(large) == ((False, False), (False, False), (256, 2) if cached else (128, 4))
