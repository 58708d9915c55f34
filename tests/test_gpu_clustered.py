"""All-agents radius queries of clustered clouds, where the lattice's mean
density says little about a row: tiles with crowded chunks (work items made
smaller there, groups whose hits overflow the buffer, rows longer than it) and
groups that overflow in the middle of a walk; bit for bit against the oracle,
and by row counts at a size where work items hold many queries."""
import numpy as np
import pytest

from gpu_util import assert_same, say
from stash_lists import lists

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_cs_0608108_amd import sphidx
    sphidx.load()
    return sphidx


def _cloud(rng, log2, F, n, clusters, sigma):
    W = [1 << (log2[a] + F) for a in range(3)]
    member = rng.integers(0, clusters, n)
    pts = []
    for a in range(3):
        centre = rng.integers(0, W[a], clusters)
        pts.append(((centre[member] + np.rint(rng.normal(0, sigma * (1 << F), n)).astype(np.int64)) % W[a]).astype(np.uint32))
    for a in range(3):
        pts[a][: n // 4] = rng.integers(0, W[a], n // 4)  # a sparse background
    return tuple(pts)


# mean rows of 12 pairs and more go by tiles, below by groups; the rows of a
# cluster's middle are several to hundreds of times longer
@pytest.mark.parametrize("mask", [7, 0])
@pytest.mark.parametrize("n, clusters, sigma, rc, tiles", [
    (20000, 15, 1.5, 2.0, True),
    (16500, 3, 0.7, 2.0, True),      # rows of thousands
    (20000, 6, 1.5, 1.2, False),
    (16500, 3, 0.7, 1.3, False),
])
def test_clustered_rows_match_oracle(sx, orc, n, clusters, sigma, rc, tiles, mask):
    import torch
    log2, F = (5, 5, 5), 14
    pts = _cloud(np.random.default_rng(n + clusters + mask), log2, F, n, clusters, sigma)
    r = int(rc * (1 << F))
    lat = sx.Lattice(log2, F, mask, n)
    dev = tuple(sx.to_dev_u32(p) for p in pts)
    lat.build(*dev)
    tab = sx.Tables(lat, 2, r)
    g = orc.Grid(orc.Lattice(log2, F, mask), pts)
    ref = g.radius(r)
    g.close()
    lens = np.diff(ref.row_ptr)
    assert lens.max() > 256 and (clusters > 3 or lens.max() > 960)
    q = sx.make_queries(n, None, r)
    for cap in (64, 256):
        for grouped in (0, 1):
            for stash in (True, False):
                say(f"clustered n={n} r={rc} mask={mask} cap={cap} grouped={grouped} stash={stash}")
                ln = sx.LaunchConfig(grouped=grouped, interior=1, sort_cap=cap)
                buf = sx.QueryBuffers(n, len(ref.ids), stash_pairs=len(ref.ids) if stash else 0)
                sx.count(lat, tab, q, buf, ln)
                assert lists(buf)["tiles"] == (tiles and stash)
                sx.write(lat, tab, q, buf, ln)
                torch.cuda.synchronize()
                assert_same(buf.host(), ref, f"cap {cap} grouped {grouped} stash {stash}")


def test_crowded_chunks_make_more_items(sx):
    """One wavefront is not left with the queries of a crowded chunk in few
    items: each holds the fewer of them, the more the chunk has."""
    import torch
    lg, F, n = 7, 16, 1 << 20
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    W = 1 << (lg + F)
    pts = [torch.randint(0, W, (n,), dtype=torch.int32, device="cuda", generator=gen) for _ in range(3)]
    lat = sx.Lattice((lg,) * 3, F, 7, n)
    tab = sx.Tables(lat, 2, 2 << F)
    q = sx.make_queries(n, None, 2 << F)
    buf, plain = sx.QueryBuffers(n, 0, want_dist2=False, stash_pairs=1 << 25), sx.QueryBuffers(n, 0, want_dist2=False)
    items = []
    for crowded in (False, True):
        if crowded:  # a quarter of the agents in a ball of some cells
            for p in pts:
                p[: n // 4] = (W // 2 + torch.randn(n // 4, device="cuda", generator=gen) * (4 << F)).int()
        lat.build(*pts)
        sx.count(lat, tab, q, buf, sx.LaunchConfig(grouped=1, interior=1))
        sx.count(lat, tab, q, plain, sx.LaunchConfig(schedule=sx.SCHED_PLAIN))
        assert torch.equal(buf.row_ptr, plain.row_ptr)
        left = lists(buf)
        assert left["tiles"]
        items.append(left["items"])
    # the crowded quarter goes by 16 queries an item
    assert items[1] > 0.8 * (n // 4 // 16) + 0.6 * items[0], items
