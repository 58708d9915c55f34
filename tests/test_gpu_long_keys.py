"""Long radius rows whose (dist^2, id) does not pack into 64 bits (fine
fractions, many objects): counted, ordered and kept in one walk like the
others, below and past the block's 3,072 pairs; bit for bit against the
oracle."""
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


# fraction bits of a cell: with ids of 16 bits and radii up to 6 cells, keys
# that pack, that pack for the shorter rows only, and that never do (in the
# last, no more than one distance bucket's span packs with an id)
@pytest.mark.parametrize("frac, mask", [(20, 7), (22, 0), (23, 7), (26, 0)])
@pytest.mark.parametrize("waves", [2, 4, 8])
def test_long_rows_of_wide_keys(sx, orc, frac, mask, waves):
    import torch
    log2 = (4, 4, 4)
    E, W = 1 << frac, 16 << frac
    n = 40000  # about 10 objects per cell
    rng = np.random.default_rng(900 + frac)
    pts = [rng.integers(0, W, n).astype(np.uint32) for _ in range(3)]
    for a in range(3):
        pts[a][:500] = 5 * E + 12345            # objects at one place
        pts[a][500:4000] = 11 * E + 777         # more than a shell holds
    pts = tuple(pts)
    lat = lattice(sx, log2, frac, mask, pts, cell_list=False)
    rmax = min(6 * E, (1 << 31) - (4 << frac))
    tab = sx.Tables(lat, 1, rmax)
    Qn = 150
    cen = [rng.integers(0, W, Qn).astype(np.uint32) for _ in range(3)]
    r = np.minimum(rng.integers(2 * E, 6 * E, Qn), rmax).astype(np.uint32)
    for a in range(3):
        cen[a][:4] = 5 * E + 12345
        cen[a][4:8] = 11 * E + 777
    r[:8] = np.minimum([0, 1, E, 5 * E, 0, 1, E, 5 * E], rmax)
    cen = tuple(cen)
    g = orc.Grid(orc.Lattice(log2, frac, mask), pts)
    ref = g.radius(r, queries=cen)
    g.close()
    lens = np.diff(ref.row_ptr)
    assert ((lens > 256) & (lens <= 3072)).sum() > 30 and (lens > 3072).sum() > 5
    keep = tuple(sx.to_dev_u32(c) for c in cen) + (sx.to_dev_u32(r),)
    q = sx.make_queries(Qn, keep[:3], keep[3])
    for method in (sx.METHOD_SPHERE, sx.METHOD_CUBE):
        for stash, d2 in ((True, True), (True, False), (False, True)):
            say(f"wide keys frac={frac} mask={mask} waves={waves} method={method} stash={stash} d2={d2}")
            ln = sx.LaunchConfig(method=method, long_row_waves=waves)
            buf = sx.QueryBuffers(Qn, int(ref.row_ptr[-1]), want_dist2=d2, stash_pairs=len(ref.ids) if stash else 0)
            sx.count(lat, tab, q, buf, ln)
            if stash and method == sx.METHOD_SPHERE:
                # every row that the block counts (expected past 5/4 of a
                # wavefront's 256) and that fits its buffer is kept
                by_block = 4.18879 * (r / E) ** 3 * n / 4096 > 1.25 * 256
                left = lists(buf)
                assert left["walk"] + left["big"] <= ((lens > 3072) | ((lens > 256) & ~by_block)).sum(), left
            sx.write(lat, tab, q, buf, ln)
            torch.cuda.synchronize()
            assert_same(buf.host(), ref, f"frac {frac}, waves {waves}, method {method}")
    code, flags = lat.status()
    assert code == sx.OK, (code, flags)
