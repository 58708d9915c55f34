"""grouped = 2: one query per wavefront where the library's choice (grouped =
0) would take groups or tiles; rows as the oracle's, and no list or item of a
grouped count."""
import numpy as np
import pytest

from gpu_util import assert_same, lattice, say
from stash_lists import lists

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_cs_0608108_amd import sphidx
    sphidx.load()
    return sphidx


@pytest.mark.parametrize("mask", [7, 0])
def test_one_query_per_wavefront_on_request(sx, orc, mask):
    import torch
    rng = np.random.default_rng(1500 + mask)
    log2, F, n = (5, 5, 5), 12, 66000
    pts = tuple(rng.integers(0, 32 << F, n).astype(np.uint32) for _ in range(3))
    lat = lattice(sx, log2, F, mask, pts, cell_list=False)
    tab = sx.Tables(lat, 2, 4 << F)
    r = 3 << (F - 1)
    g = orc.Grid(orc.Lattice(log2, F, mask), pts)
    ref = g.radius(r)
    refk = g.knn(np.full(n, 20, np.uint32), np.full(n, 4 << F, np.uint32))
    g.close()
    for mode, want in ((sx.MODE_RADIUS, ref), (sx.MODE_KNN, refk)):
        q = sx.make_queries(n, None, r if mode == sx.MODE_RADIUS else 4 << F, 20, mode)
        for grouped in (0, 2):
            say(f"one per wavefront mask={mask} mode={mode} grouped={grouped}")
            ln = sx.LaunchConfig(grouped=grouped, interior=1)
            buf = sx.QueryBuffers(n, len(want.ids), stash_pairs=len(want.ids))
            sx.count(lat, tab, q, buf, ln)
            left = lists(buf)
            sx.write(lat, tab, q, buf, ln)
            torch.cuda.synchronize()
            assert_same(buf.host(), want, f"mode {mode} grouped {grouped}")
            if grouped == 2:
                assert not left["tiles"] and left["items"] == 0 and left["extra"] == 0 and left["long"] == 0, left
            elif mode == sx.MODE_RADIUS:
                assert left["tiles"] and left["items"] > 0, left
            else:
                assert left["extra"] > 0, left  # rows short of K inside their first radius
    with pytest.raises(sx.SphidxError):
        sx.count(lat, tab, q, buf, sx.LaunchConfig(grouped=3))
