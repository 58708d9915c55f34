"""The stash copy's shapes: a group of rows shared by several wavefronts (few
rows), one row per wavefront, and up to 64 rows per wavefront, at the batch
sizes where the shape changes; rows of no, few and thousands of pairs, bit for
bit against the oracle."""
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
    rng = np.random.default_rng(900)
    log2, F, n = (4, 4, 4), 10, 12000
    pts = tuple(rng.integers(0, 16 << F, n).astype(np.uint32) for _ in range(3))
    lat = lattice(sx, log2, F, 0, pts)
    tab = sx.Tables(lat, 2, 6 << F)
    return sx, lat, tab, orc.Grid(orc.Lattice(log2, F, 0), pts)


@pytest.mark.parametrize("q", [1, 2, 1024, 1025, 2049, 4097, 8192, 8193, 16385, 33001])
@pytest.mark.parametrize("d2", [True, False])
def test_copy_shapes_match_oracle(world, q, d2):
    sx, lat, tab, g = world
    rng = np.random.default_rng(q)
    cen = tuple(rng.integers(0, 16 << 10, q).astype(np.uint32) for _ in range(3))
    r = rng.integers(0, 1 << 10, q).astype(np.uint32)  # short and empty rows
    r[rng.integers(0, q, 1 + q // 200)] = 6 << 10      # and rows of up to 2,600 pairs
    ref = g.radius(r, queries=cen)
    say(f"stash copy, {q} rows, {len(ref.ids)} pairs, dist2 {d2}")
    got = run(sx, lat, tab, r, queries=cen, want_dist2=d2, stash=True)
    assert_same(got, ref, f"{q} rows")
