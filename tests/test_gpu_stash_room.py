"""sphidx_query_stash_bytes gives the size that keeps every row: all-agents
queries counted by tiles, by groups and one per wavefront leave nothing to the
write pass, over batch sizes at which the waves' chunks are small or large
against the rows of one tile group."""
import pytest

from gpu_util import say
from stash_lists import lists

pytestmark = pytest.mark.gpu

F = 16


@pytest.fixture(scope="module")
def sx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_cs_0608108_amd import sphidx
    sphidx.load()
    return sphidx


@pytest.mark.parametrize("mask", [7, 0])
@pytest.mark.parametrize("lg, n, rc, tiles", [
    (5, 1024, 5.0, True),       # the smallest batch the tiles take
    (5, 16384, 2.5, True),
    (6, 100003, 2.5, True),
    (6, 250007, 2.0, True),
    (7, 524288, 3.0, True),
    (7, 1 << 20, 2.5, True),    # a grab holds one group's rows or two
    (7, 1 << 20, 3.0, True),
    (7, 1 << 21, 2.5, True),
    (7, 1 << 20, 1.5, False),   # rows below those the tiles take
])
def test_stash_bytes_keep_every_row(sx, lg, n, rc, tiles, mask):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(n + mask)
    pts = [torch.randint(0, 1 << (lg + F), (n,), dtype=torch.int32, device="cuda", generator=g) for _ in range(3)]
    lat = sx.Lattice((lg,) * 3, F, mask, n)
    lat.build(*pts)
    r = int(rc * (1 << F))
    tab = sx.Tables(lat, 2, r)
    q = sx.make_queries(n, None, r)
    plain = sx.QueryBuffers(n, 0, want_dist2=False)
    sx.count(lat, tab, q, plain, sx.LaunchConfig(schedule=sx.SCHED_PLAIN))
    total = int(plain.row_ptr[-1].item())
    for d2 in (False, True):
        for ln in (sx.LaunchConfig(grouped=1, interior=1),
                   sx.LaunchConfig(grouped=1, interior=1, tile=16, blocks_per_cu=6), sx.LaunchConfig(interior=1)):
            say(f"stash room lg={lg} n={n} r={rc} mask={mask} grouped={ln.grouped} bpc={ln.blocks_per_cu} d2={d2}")
            buf = sx.QueryBuffers(n, 0, want_dist2=d2, stash_pairs=total)
            sx.count(lat, tab, q, buf, ln)
            left = lists(buf)
            assert torch.equal(buf.row_ptr, plain.row_ptr)
            assert left["kept"] and (left["tiles"] == tiles or not ln.grouped), left
            assert left["walk"] == 0 and left["big"] == 0, (left, n, total)
            del buf
