"""Small batches: one block clears and sets up (to 1,024 queries), the main
kernels take the fallback queries (to 8,192); centres outside the region,
radii beyond the tables' cap and short of it, radius and K-NN rows mixed, rows
kept and walked again, at the sizes where the launches change; bit for bit
against the oracle."""
import numpy as np
import pytest

from gpu_util import assert_same, lattice, run, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def world(orc):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_cs_0608108_amd import sphidx as sx
    sx.load()
    rng = np.random.default_rng(1100)
    log2, F, n, mask = (4, 4, 5), 10, 6000, 4
    pts = [rng.integers(0, (1 << log2[a]) << F, n).astype(np.uint32) for a in range(3)]
    for a in range(2):
        pts[a][:300] += 16 << F  # outside the region on the clipped axes
    pts = tuple(pts)
    lat = lattice(sx, log2, F, mask, pts)
    tab = sx.Tables(lat, 2, 3 << F)
    return sx, lat, tab, orc.Grid(orc.Lattice(log2, F, mask), pts)


@pytest.mark.parametrize("q", [1, 63, 1024, 1025, 8192, 8193])
def test_small_batches_match_oracle(world, q):
    sx, lat, tab, g = world
    rng = np.random.default_rng(q)
    cen = [rng.integers(0, 16 << 10, q).astype(np.uint32) for _ in range(3)]
    cen[0][rng.random(q) < 0.1] += 16 << 10                   # centres outside
    r = rng.integers(0, 3 << 10, q).astype(np.uint32)
    r[rng.random(q) < 0.1] = 4 << 10                          # beyond the tables
    if q > 100:
        r[rng.integers(0, q, 3)] = 20 << 10                   # the whole world: rows of thousands
    k = np.where(rng.random(q) < 0.4, rng.integers(1, 100, q), 0).astype(np.uint32)
    ref, refm = g.radius(r, queries=cen), g.mixed(k, r, queries=cen)
    refk = g.mixed(np.full(q, 5, np.uint32), r, queries=cen)
    for ln in (sx.LaunchConfig(), sx.LaunchConfig(grouped=1, sort_cap=128), sx.LaunchConfig(schedule=sx.SCHED_PLAIN)):
        for stash in (False, True):
            say(f"small batch {q} grouped {ln.grouped} schedule {ln.schedule} stash {stash}")
            assert_same(run(sx, lat, tab, r, queries=cen, launch=ln, stash=stash), ref, "radius")
            assert_same(run(sx, lat, tab, r, k=k, mode=sx.MODE_MIXED, queries=cen, launch=ln, stash=stash), refm, "mixed")
            assert_same(run(sx, lat, tab, r, k=5, mode=sx.MODE_KNN, queries=cen, launch=ln, stash=stash), refk, "knn")
    code, flags = lat.status()
    assert code == sx.OK, (code, flags)


@pytest.mark.parametrize("n", [16383, 16384, 40001])
def test_default_launch_of_all_agents_batches(orc, n):
    """Either side of the size from which the library takes them in groups."""
    from paper_cs_0608108_amd import sphidx as sx
    rng = np.random.default_rng(n)
    log2, F, mask = (5, 5, 5), 12, 3
    pts = tuple(rng.integers(0, 32 << F, n).astype(np.uint32) for _ in range(3))
    pts[2][:50] += 32 << F
    lat = lattice(sx, log2, F, mask, pts)
    tab = sx.Tables(lat, 2, 4 << F)
    g = orc.Grid(orc.Lattice(log2, F, mask), pts)
    r = rng.integers(0, 2 << F, n).astype(np.uint32)
    cap = np.full(n, 4 << F, np.uint32)
    k = np.where(rng.random(n) < 0.5, rng.integers(1, 20, n), 0).astype(np.uint32)
    rm = np.where(k > 0, cap, r).astype(np.uint32)
    cases = [("radius", 2 << F, None, sx.MODE_RADIUS, g.radius(2 << F)), ("uneven", r, None, sx.MODE_RADIUS, g.radius(r)),
             ("knn", 4 << F, 10, sx.MODE_KNN, g.mixed(np.full(n, 10, np.uint32), cap)),
             ("mixed", rm, k, sx.MODE_MIXED, g.mixed(k, rm))]
    for what, rr, kk, mode, ref in cases:
        for stash in (False, True):
            say(f"default launch n {n} {what} stash {stash}")
            assert_same(run(sx, lat, tab, rr, k=kk, mode=mode, stash=stash), ref, what)
