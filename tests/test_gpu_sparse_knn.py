"""All-agents K-NN by the default launch where the lattice's mean density is
low: one query per wavefront or groups by a sample of the objects, uniform
clouds and clusters in a sparse background, one K or a K per query, at the
lattice's edges and with objects outside; bit for bit against the oracle, and by
the lists that the count pass leaves."""
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


# (log2 cells, mask, objects in clusters of the whole, K or None for a K per
# query, whether the batch goes in groups)
@pytest.mark.parametrize("log2, mask, clustered, k, groups", [
    ((7, 6, 7), 7, 0.0, 12, False),        # 0.063 objects per cell
    ((7, 6, 7), 0, 0.0, None, False),
    ((7, 6, 7), 0, 0.6, 12, True),
    ((7, 6, 7), 7, 0.6, None, True),
    ((7, 6, 7), 7, 0.0, 1, None),          # K = 1: in groups, each its own nearest: no list shows it
    ((5, 6, 6), 0, 0.0, 12, True),         # 0.5 objects per cell
    ((6, 6, 6), 7, 0.0, 64, False),        # 0.25 per cell, too few for K = 64
    ((2, 8, 8), 2, 0.0, 40, False),        # four cells along x
])
def test_sparse_rows_match_oracle(sx, orc, log2, mask, clustered, k, groups):
    import torch
    rng = np.random.default_rng(77 + mask)
    F, n = 12, 66001
    W = [1 << (log2[a] + F) for a in range(3)]
    pts = list(tiny_points(rng, log2, F, mask, n, outside=(mask == 0)))
    m = int(clustered * n)
    if m:
        centre = rng.integers(0, 20, m)
        for a in range(3):
            c = rng.integers(0, W[a], 20)[centre]
            pts[a][n // 5:n // 5 + m] = (c + rng.normal(0, 2 << F, m).astype(np.int64)) % W[a]
    pts = tuple(pts)
    lat = lattice(sx, log2, F, mask, pts, cell_list=False)
    cap = (4 if 2 in log2 else 6) << F
    tab = sx.Tables(lat, 2, cap)
    kk = rng.integers(0, 70, n).astype(np.uint32) if k is None else np.full(n, k, np.uint32)
    g = orc.Grid(orc.Lattice(log2, F, mask), pts)
    ref = g.knn(kk, np.full(n, cap, np.uint32))
    g.close()
    kd = sx.to_dev_u32(kk) if k is None else k
    q = sx.make_queries(n, None, cap, kd, sx.MODE_KNN)
    for ln in (sx.LaunchConfig(), sx.LaunchConfig(grouped=1), sx.LaunchConfig(grouped=2)):
        say(f"sparse knn {log2} mask={mask} k={k} grouped={ln.grouped}")
        buf = sx.QueryBuffers(n, len(ref.ids), stash_pairs=int(kk.sum()))
        sx.count(lat, tab, q, buf, ln)
        left = lists(buf)
        sx.write(lat, tab, q, buf, ln)
        torch.cuda.synchronize()
        assert_same(buf.host(), ref, f"grouped {ln.grouped}")
        # (a grouped count passes the fallback rows through its lists)
        alone = left["extra"] in (0, left["fallback"]) and left["long"] <= left["fallback"]
        assert groups is None or alone == (ln.grouped == 2 or (ln.grouped == 0 and not groups)), left
    del kd


@pytest.mark.parametrize("clustered", [0.0, 0.7])
def test_sampled_mixed_batches_and_replays(sx, orc, clustered):
    """A mixed batch (radius and K-NN rows) whose path the sample chooses, and
    one captured graph replayed while the objects change from sparse to
    clustered and back: every replay as the oracle has it."""
    import torch
    log2, F, n = (7, 6, 7), 12, 66000
    rng = np.random.default_rng(int(clustered * 10) + 5)
    W = [1 << (log2[a] + F) for a in range(3)]

    def cloud(share):
        pts = [rng.integers(0, W[a], n) for a in range(3)]
        m = int(share * n)
        if m:
            centre = rng.integers(0, 24, m)
            for a in range(3):
                pts[a][:m] = (rng.integers(0, W[a], 24)[centre] + rng.normal(0, 2 << F, m).astype(np.int64)) % W[a]
        return tuple(p.astype(np.uint32) for p in pts)

    cap = 5 << F
    r = np.where(np.arange(n) % 3 == 0, rng.integers(1, 2 << F, n), cap).astype(np.uint32)
    k = np.where(np.arange(n) % 3 == 0, 0, rng.integers(1, 40, n)).astype(np.uint32)
    rd, kd = sx.to_dev_u32(r), sx.to_dev_u32(k)
    lat = sx.Lattice(log2, F, 7, n)
    tab = sx.Tables(lat, 1, cap)
    dev = [sx.to_dev_u32(p) for p in cloud(clustered)]
    q = sx.make_queries(n, None, rd, kd, sx.MODE_MIXED)
    buf = sx.QueryBuffers(n, 4_000_000, stash_pairs=4_000_000)
    lat.build(*dev)
    name = sx.count_kernel(lat, tab, q, buf)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        lat.build(*dev)
        sx.query(lat, tab, q, buf)
        side.synchronize()
        with torch.cuda.graph(graph, stream=side):
            lat.build(*dev)
            sx.query(lat, tab, q, buf)
    torch.cuda.synchronize()
    for share in (clustered, 0.7 - clustered, clustered, 0.7 - clustered):
        pts = cloud(share)
        for d, p in zip(dev, pts):
            d.copy_(sx.to_dev_u32(p))
        graph.replay()
        torch.cuda.synchronize()
        g = orc.Grid(orc.Lattice(log2, F, 7), pts)
        ref = g.mixed(k, r)
        g.close()
        assert len(ref.ids) <= 4_000_000
        say(f"sampled mixed replay share={share} kernel={name} pairs={len(ref.ids)}")
        assert_same(buf.host(), ref, f"share {share}")
    del rd, kd
