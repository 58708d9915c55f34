"""sphidx_count_kernel names the kernel that the count pass takes, as seen by
the lists that it leaves: tiles, groups, one query per wavefront, and what the
launch, the batch and its size change; NULL for a refused call."""
import numpy as np
import pytest

from gpu_util import lattice
from stash_lists import lists

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_cs_0608108_amd import sphidx
    sphidx.load()
    return sphidx


def test_count_kernel_names(sx):
    rng = np.random.default_rng(4)
    log2, F, n = (5, 5, 5), 12, 70000
    E = 1 << F
    pts = tuple(rng.integers(0, 32 << F, n).astype(np.uint32) for _ in range(3))
    lat = lattice(sx, log2, F, 7, pts, cell_list=False)
    wide, tab2 = sx.Tables(lat, 2, 4 * E), sx.Tables(lat, 2, 2 * E)
    cen = tuple(sx.to_dev_u32(p[:5000]) for p in pts)
    uneven = sx.to_dev_u32(rng.integers(E // 2, 2 * E, n).astype(np.uint32))
    one = sx.make_queries(n, None, 2 * E)            # rows of some 70 pairs
    few = sx.make_queries(n, None, E // 2)           # of one
    each = sx.make_queries(n, None, uneven)
    knn = sx.make_queries(n, None, 4 * E, 10, sx.MODE_KNN)
    some = sx.make_queries(5000, cen, 2 * E)
    T, G, C = "tile_count_kernel", "group_count_kernel", "count_kernel"
    L = sx.LaunchConfig
    plain = L(schedule=sx.SCHED_PLAIN)
    for q, ln, stash, want in [
        (one, L(), True, T), (one, L(grouped=1), True, T), (one, L(grouped=2), True, C), (one, plain, True, C),
        (few, L(), True, G), (each, L(), True, G), (each, L(grouped=2), True, C), (knn, L(), True, G),
        (knn, L(), False, C), (knn, L(grouped=1, interior=1), False, G), (some, L(), True, C), (some, L(grouped=1), True, G),
        (one, L(method=sx.METHOD_PAPER64), True, C), (one, L(method=sx.METHOD_CUBE, grouped=1), True, G),
        (one, L(grouped=3), True, None), (one, L(sort_cap=100), True, None),
    ]:
        tab = wide if q is knn else tab2
        buf = sx.QueryBuffers(q.count, 0, want_dist2=False, stash_pairs=70000 * 120 if stash else 0)
        assert sx.count_kernel(lat, tab, q, buf, ln) == want, (ln, want)
        if want is None:
            with pytest.raises(sx.SphidxError):
                sx.count(lat, tab, q, buf, ln)
            continue
        sx.count(lat, tab, q, buf, ln)
        left = lists(buf)
        assert (left["items"] > 0) == (want == T), (want, left)
        if stash:
            assert left["tiles"] == (want == T), (want, left)
    del uneven, cen


def test_tile_worlds_go_by_tiles(sx):
    """The worlds that the tile kernel's rows are compared with the oracle on
    are counted by it."""
    from test_gpu_tiles import WORLDS, _lat, _points
    for world, (log2, F, mask, n, rc) in enumerate(WORLDS):
        pts = _points(np.random.default_rng(40 + world), world)
        r = int(rc * (1 << F))
        lat = _lat(sx, log2, F, mask, pts, xorder=(world % 2 == 1))
        tab = sx.Tables(lat, 2, r)
        q = sx.make_queries(n, None, r)
        for stash in (0, 1 << 24):
            buf = sx.QueryBuffers(n, 0, stash_pairs=stash)
            assert sx.count_kernel(lat, tab, q, buf, sx.LaunchConfig(grouped=1, interior=1)) == "tile_count_kernel", world
