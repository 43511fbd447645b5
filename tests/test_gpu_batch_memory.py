"""Device memory that a batch keeps: the tile lists of sparse items are of their
tiles, not of every tile that their cells could hold."""
import numpy as np
import pytest

import oracle
import paper_1210_1833_amd as cute

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible: the gpu tests need an MI355X")
    cute.load()
    yield


def test_many_sparse_items():
    import torch
    # 900 points in 36^3 cells: about 900 tiles, and cells for 46 700
    a = np.random.default_rng(9).uniform(0.0, 3600.0, (900, 3))
    e = np.linspace(0.0, 100.0, 5)
    bn, ob = cute.Binning(cute.BIN_MONO, e), oracle.Binning(oracle.MONO, e)
    g = cute.build_grid(a, cute.GEOM_BOX_OPEN, r_max=100.0, cell_size=100.0)
    items = [cute.BatchItem(g, None, bn) for _ in range(1000)]
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    b = cute.Batch(items)
    used = before - torch.cuda.mem_get_info()[0]
    print("batch of 1000 sparse items: %.1f MB" % (used / 1e6), flush=True)
    b.run()
    got = b.counts()
    want = oracle.count_pairs(a, None, ob)
    np.testing.assert_array_equal(np.asarray(got).reshape(1000, -1), np.tile(want, (1000, 1)))
    assert used < 200e6   # (750 MB of slots before; the library's pool may hold 256 MB already)
