"""Element tiles around a particle of many corners end where their LDS does, not where a
corner code's rank does: such a particle takes further entries in its tile, which no
caller of the plan sees."""
import numpy as np
import pytest

from fans import disc, tet_fan
from paper_2104_02646_amd import gsim as G
from paper_2104_02646_amd import workloads as W


def loose(n):
    X = np.concatenate([np.array([[0, 0, 0], [1, 0, 0], [0, 1, 0], [0, 0, 1.0]]) + [2.0 * k, 0, 0] for k in range(n)])
    return W.Body(X=X, tets=np.arange(4 * n, dtype=np.int32).reshape(-1, 4), mu=np.ones(n), lam=np.ones(n),
                  mass=np.ones(4 * n))


@pytest.mark.parametrize("tile", [0, 32, 512, 2048])
@pytest.mark.parametrize("body", [lambda: tet_fan(33), lambda: tet_fan(1500), lambda: disc(700), lambda: disc(700, True),
                                  lambda: loose(800)], ids=["fan 33", "fan 1500", "disc", "disc with air", "loose"])
def test_tiles_end_at_their_lds(body, tile):
    import torch
    b = body()
    p = G.Plan([b], torch.float32, tile)
    tiles, tp, run, slot = p.tiles()
    limit = tile or 256
    want = []
    for kind, idx in ((0, b.tets), (1, b.tris), (2, b.hinges)):
        nc = 3 if kind == 1 else 4
        wp, wc = (12, 8) if kind == 1 and b.air else (8, 4)
        e = 0
        while e < len(idx):
            n, seen = 0, set()
            while e + n < len(idx) and n < limit:
                more = seen | set(map(int, idx[e + n]))
                if n and wp * len(more) + wc * nc * (n + 1) > 16384:
                    break
                seen, n = more, n + 1
            want.append((kind, e, n, sorted(seen)))
            e += n
    ends = list(tiles[1:, 4]) + [len(tp)]
    got = [(int(t[0]), int(t[2]), int(t[3]), tp[t[4]:ends[i]].tolist()) for i, t in enumerate(tiles)]
    assert got == want
    assert sorted(slot.tolist()) == sorted(set(slot.tolist())) and (run >> 16).min() >= 1
    for i, (kind, e, n, parts) in enumerate(want):  # every run holds the particle's corners of the tile
        idx = (b.tets, b.tris, b.hinges)[kind][e:e + n].ravel()
        assert (run[tiles[i, 4]:ends[i]] >> 16).tolist() == [int((idx == q).sum()) for q in parts]
