"""Cell starts of a rebuilt lattice at the sizes where its prefix sum changes
shape: one block (up to four chunks of 4,096 counts), block totals added up by
the blocks behind them (to 8,192 blocks), totals scanned in between."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("log2", [(4, 5, 4), (5, 5, 4), (6, 5, 7), (8, 8, 8), (9, 8, 8)])
def test_cell_starts(log2):
    import torch
    from paper_cs_0608108_amd import sphidx
    F, n = 8, 50000
    rng = np.random.default_rng(sum(log2))
    pts = [rng.integers(0, 1 << (lg + F), n, dtype=np.uint32) for lg in log2]
    for a, lg in enumerate(log2):  # the first and the last cells hold objects
        pts[a][:5], pts[a][5:9] = 0, (1 << (lg + F)) - 1
    lat = sphidx.Lattice(log2, F, 7, n)
    dev = tuple(sphidx.to_dev_u32(a) for a in pts)
    cell = [p.astype(np.int64) >> F for p in pts]
    packed = (cell[2] << (log2[0] + log2[1])) | (cell[1] << log2[0]) | cell[0]
    want = torch.zeros(lat.ncells + 3, dtype=torch.int64)
    want[1:] = torch.cumsum(torch.bincount(torch.from_numpy(packed), minlength=lat.ncells + 2), 0)
    off = lat.view().cell_start - lat.workspace.data_ptr()
    for _ in range(2):
        print("scan", log2, flush=True)
        lat.build(*dev)
        got = lat.workspace[off:off + 4 * (lat.ncells + 3)].view(torch.int32).cpu()
        assert torch.equal(got.long(), want)
