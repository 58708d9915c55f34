"""Grouped count of mixed radii and K-NN rows: candidate streams shorter and
longer than one window of row marks (256 slots), rows that end inside, at and
past a 64-slot step, empty rows, one query per group up to eight, K-NN groups
held by their expected hits rather than their rows, with and without a stash
and distances; bit for bit against the oracle."""
import numpy as np
import pytest

from gpu_util import assert_same, run, say, tiny_points

pytestmark = pytest.mark.gpu

# world, fraction bits, mask, objects, largest radius in cells, K, cap in cells
WORLDS = [
    ((4, 4, 4), 16, 7, 2 * 4096, 3.0, 10, 5.0),    # streams of some steps
    ((5, 5, 5), 16, 0, 3001, 6.0, 10, 12.0),       # sparse: rows far past the hits, objects outside
    ((3, 3, 3), 12, 7, 30000, 1.0, 16, 2.0),       # 59 objects per cell: windows of marks
    ((4, 3, 5), 10, 2, 64, 2.0, 1, 4.0),           # empty rows almost everywhere
    ((6, 4, 5), 14, 5, 20011, 4.0, 40, 6.0),
]


@pytest.fixture(scope="module")
def sx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_cs_0608108_amd import sphidx
    sphidx.load()
    return sphidx


@pytest.mark.parametrize("xorder", [False, True])
@pytest.mark.parametrize("world", range(len(WORLDS)))
def test_grouped_rows_match_oracle(sx, orc, world, xorder):
    log2, F, mask, n, rc, k, cap = WORLDS[world]
    rng = np.random.default_rng(900 + world)
    pts = tiny_points(rng, log2, F, mask, n, outside=(mask != 7), invalid=(mask != 7))
    lat = sx.Lattice(log2, F, mask, n)
    if xorder:
        lat.set_cell_order(sx.ORDER_X)
    dev = tuple(sx.to_dev_u32(a) for a in pts)
    lat.build(*dev)
    g = orc.Grid(orc.Lattice(log2, F, mask), pts)
    e = 1 << F
    r = rng.integers(1, int(rc * e) + 1, n).astype(np.uint32)
    r[::7] = int(rc * e)
    rcap = int(cap * e)
    ks = rng.integers(1, k + 1, n).astype(np.uint32)
    tab = sx.Tables(lat, 2, max(rcap, int(rc * e)))
    for flags in (0, sx.EXCLUDE_SELF):
        radius, near = g.radius(r, flags=flags), g.knn(ks, rcap, flags=flags)
        for cap_rows, stash, d2 in ((256, True, True), (256, False, True), (64, True, False)):
            ln = sx.LaunchConfig(grouped=1, sort_cap=cap_rows)
            say(f"groups world {world} xorder {xorder} flags {flags} sort_cap {cap_rows} stash {stash}")
            assert_same(run(sx, lat, tab, r, flags=flags, launch=ln, want_dist2=d2, stash=stash), radius, "radius")
            assert_same(run(sx, lat, tab, rcap, ks, sx.MODE_KNN, flags=flags, launch=ln, want_dist2=d2, stash=stash),
                        near, "nearest")
    g.close()
