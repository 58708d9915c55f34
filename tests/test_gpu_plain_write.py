"""Rows counted by tiles and written by the plain schedule: rows that the stash
has no room for, rows kept without the distances that the write asks for, rows
all kept, and objects outside the region, with per-query walks (sphere tables,
the per-query choice) in the write's launch; bit for bit against the oracle."""
import numpy as np
import pytest

from gpu_util import assert_same, say, tiny_points
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
@pytest.mark.parametrize("n", [1030, 9001])
@pytest.mark.parametrize("frac", [1.0, 0.3])
def test_plain_write_after_tiles(sx, orc, mask, n, frac):
    import torch
    log2, F = ((4, 4, 4), 12) if n < 4096 else ((5, 5, 5), 12)
    pts = tiny_points(np.random.default_rng(n + mask), log2, F, mask, n, outside=(mask == 0), invalid=(mask == 0))
    r = (5 << F) // 2
    lat = sx.Lattice(log2, F, mask, n)
    dev = tuple(sx.to_dev_u32(p) for p in pts)
    lat.build(*dev)
    tab = sx.Tables(lat, 2, r)
    g = orc.Grid(orc.Lattice(log2, F, mask), pts)
    ref = g.radius(r)
    g.close()
    total = len(ref.ids)
    q = sx.make_queries(n, None, r)
    for launch in (sx.LaunchConfig(schedule=sx.SCHED_PLAIN), sx.LaunchConfig(schedule=sx.SCHED_PLAIN, sort_cap=64, tile=3)):
        say(f"plain write after tiles mask={mask} n={n} frac={frac} cap={launch.sort_cap}")
        buf = sx.QueryBuffers(n, total, want_dist2=False, stash_pairs=int(total * frac))
        sx.count(lat, tab, q, buf, sx.LaunchConfig(grouped=1, interior=1))
        left = lists(buf)
        assert left["tiles"], left
        sx.write(lat, tab, q, buf, launch)
        torch.cuda.synchronize()
        assert_same(buf.host(), ref, "ids")
        buf.dist2 = torch.empty(total, dtype=torch.int64, device="cuda")
        for _ in range(2):
            sx.write(lat, tab, q, buf, launch)
            torch.cuda.synchronize()
            assert_same(buf.host(), ref, "distances after a count without them")
