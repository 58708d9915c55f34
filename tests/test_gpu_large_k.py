"""All-agents K-NN with a K per query, by the default launch and in groups: K
on both sides of half the grouped kernel's buffer (rows past it go straight to
the one-query-per-wave kernel), K = 0, K past every object and K that a factor
of two would wrap; bit for bit against the oracle."""
import numpy as np
import pytest

from gpu_util import assert_same, lattice, say, tiny_points
from stash_lists import lists

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_cs_0608108_amd import sphidx
    sphidx.load()
    return sphidx


@pytest.mark.parametrize("mask", [7, 1])
@pytest.mark.parametrize("cap", [128, 256])
def test_large_k_rows_match_oracle(sx, orc, mask, cap):
    import torch
    rng = np.random.default_rng(1200 + mask + cap)
    log2, F = (5, 5, 4), 10
    n = 16500
    pts = tiny_points(rng, log2, F, mask, n, outside=(mask != 7))
    r = 4 << F
    ks = np.array([0, 1, 16, cap // 4, cap // 2 - 1, cap // 2, cap // 2 + 1, cap, 300, 5000], dtype=np.uint32)
    k = ks[rng.integers(0, len(ks), n)]
    k[5], k[6] = 1 << 31, (1 << 32) - 1
    lat = lattice(sx, log2, F, mask, pts, cell_list=False)
    tab = sx.Tables(lat, 2, r)
    g = orc.Grid(orc.Lattice(log2, F, mask), pts)
    ref = g.knn(k, np.full(n, r, np.uint32))
    g.close()
    kd = sx.to_dev_u32(k)
    q = sx.make_queries(n, None, r, kd, sx.MODE_KNN)
    for grouped in (0, 1):
        for d2 in (False, True):
            say(f"large K mask={mask} cap={cap} grouped={grouped} d2={d2}")
            ln = sx.LaunchConfig(grouped=grouped, sort_cap=cap)
            buf = sx.QueryBuffers(n, len(ref.ids), want_dist2=d2, stash_pairs=len(ref.ids))
            sx.count(lat, tab, q, buf, ln)
            left = lists(buf)
            sx.write(lat, tab, q, buf, ln)
            torch.cuda.synchronize()
            assert_same(buf.host(), ref, f"grouped {grouped}")
            assert left["kept"] and left["big"] > 0
    del kd


@pytest.mark.parametrize("mask", [7, 0])
def test_large_k_rows_pass_no_grouped_round(sx, mask):
    """Rows of K past half the buffer are on no list of the grouped rounds."""
    rng = np.random.default_rng(1300 + mask)
    log2, F, n = (5, 5, 5), 10, 20000
    pts = tuple(rng.integers(0, 32 << F, n).astype(np.uint32) for _ in range(3))
    lat = lattice(sx, log2, F, mask, pts, cell_list=False)
    tab = sx.Tables(lat, 2, 6 << F)
    k = np.full(n, 129, np.uint32)
    k[::7] = 250
    kd = sx.to_dev_u32(k)
    q = sx.make_queries(n, None, 6 << F, kd, sx.MODE_KNN)
    buf = sx.QueryBuffers(n, 0, want_dist2=False, stash_pairs=int(k.sum()))
    sx.count(lat, tab, q, buf, sx.LaunchConfig(grouped=1))
    left = lists(buf)
    assert left["extra"] == 0 and left["long"] == n, left
    del kd
