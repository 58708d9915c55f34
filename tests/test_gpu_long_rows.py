"""Long radius rows in the write pass: rows longer than the wavefront's LDS
row buffer taken by one block of 2, 4 or 8 waves (walked once, ordered by a
block-wide bucket sort), rows beyond the block's 3,072 pairs and K-NN rows
left to the windowed top-M kernel; bit for bit against the oracle, with
every walk (sphere tables, cube, per-query choice, the paper's tables)."""
import numpy as np
import pytest

from gpu_util import assert_same, lattice, run, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_cs_0608108_amd import sphidx
    sphidx.load()
    return sphidx


@pytest.mark.parametrize("mask", [7, 0])
def test_long_rows_by_block_match_oracle(sx, orc, mask):
    rng = np.random.default_rng(500 + mask)
    log2, F = (5, 5, 5), 10
    E = 1 << F
    W = 32 << F
    n = 60000  # about 1.8 objects per cell
    pts = tuple(rng.integers(0, W, n).astype(np.uint32) for _ in range(3))
    lat = lattice(sx, log2, F, mask, pts)
    tab = sx.Tables(lat, 2, 8 * E)
    Qn = 3000
    cen = tuple(rng.integers(0, W, Qn).astype(np.uint32) for _ in range(3))
    # radii from short rows (sort_cap) to rows past the block's 3,072 pairs
    r = rng.integers(0, 8 * E, Qn).astype(np.uint32)
    r[:100] = 8 * E
    k = np.where(rng.random(Qn) < 0.2, rng.integers(65, 300, Qn), 0).astype(np.uint32)
    g = orc.Grid(orc.Lattice(log2, F, mask), pts)
    ref = g.radius(r, queries=cen)
    refm = g.mixed(k, r, queries=cen)
    g.close()
    lens = np.diff(ref.row_ptr)
    assert (lens > 256).sum() > 300 and (lens > 3072).sum() > 20
    for lw in (1, 2, 4, 8):
        for method in (sx.METHOD_SPHERE, sx.METHOD_CUBE, sx.METHOD_AUTO, sx.METHOD_PAPER64):
            for stash in (False, True):
                say(f"long rows mask={mask} waves={lw} method={method} stash={stash}")
                ln = sx.LaunchConfig(method=method, long_row_waves=lw)
                assert_same(run(sx, lat, tab, r, queries=cen, launch=ln, stash=stash), ref,
                            f"radius, waves {lw}, method {method}")
        ln = sx.LaunchConfig(long_row_waves=lw, sort_cap=128)
        assert_same(run(sx, lat, tab, r, k=k, mode=sx.MODE_MIXED, queries=cen, launch=ln), refm,
                    f"mixed, waves {lw}")
    code, flags = lat.status()
    assert code == sx.OK, (code, flags)


@pytest.mark.parametrize("lw", [2, 4, 8])
@pytest.mark.parametrize("mask", [0, 7])
def test_rows_past_the_block_buffer_match_oracle(sx, orc, mask, lw):
    """Rows of 3,073 pairs and more, walked twice and ordered shell by shell:
    crowded cells, rows one pair either side of the block's buffer and of a
    shell, an object's own row left out, and shells that cannot be cut
    (thousands of objects at one distance, at radius 0 too)."""
    rng = np.random.default_rng(700 + mask)
    log2, F = (4, 4, 4), 12
    E, W = 1 << F, 16 << F
    n = 60000
    pts = [rng.integers(0, W, n).astype(np.uint32) for _ in range(3)]
    # clumps at one place of 2,560, 2,561, 3,072, 3,073 and 7,000 objects
    at = 0
    clumps = (2560, 2561, 3072, 3073, 7000)
    for i, m in enumerate(clumps):
        for a in range(3):
            pts[a][at:at + m] = 2 * E + i * 2 * E + 77
        at += m
    pts = tuple(pts)
    lat = lattice(sx, log2, F, mask, pts, cell_list=False)
    tab = sx.Tables(lat, 2, 7 * E)
    Qn = 120
    cen = [rng.integers(0, W, Qn).astype(np.uint32) for _ in range(3)]
    r = rng.integers(4 * E, 7 * E, Qn).astype(np.uint32)
    for i in range(len(clumps)):
        for j, rr in enumerate((0, 1, 3 * E)):  # the clump alone, and with its surroundings
            for a in range(3):
                cen[a][3 * i + j] = 2 * E + i * 2 * E + 77
            r[3 * i + j] = rr
    cen = tuple(cen)
    g = orc.Grid(orc.Lattice(log2, F, mask), pts)
    ref = g.radius(r, queries=cen)
    g.close()
    lens = np.diff(ref.row_ptr)
    assert (lens > 3072).sum() > 60 and (lens == 3073).any()
    for method in (sx.METHOD_SPHERE, sx.METHOD_CUBE, sx.METHOD_PAPER64):
        for stash, d2 in ((False, True), (True, False)):
            say(f"rows past the block buffer mask={mask} waves={lw} method={method} stash={stash}")
            ln = sx.LaunchConfig(method=method, long_row_waves=lw)
            assert_same(run(sx, lat, tab, r, queries=cen, launch=ln, stash=stash, want_dist2=d2), ref,
                        f"waves {lw}, method {method}")
