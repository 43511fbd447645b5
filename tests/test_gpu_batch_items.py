"""Batched counts whose workgroups move from item to item: exact against the
oracle for one item, more items than a workgroup looks through at once, empty
items among them, and items of very unequal size."""
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


SIZES = {"one": [3001], "two": [1, 900], "many": [7 * (k % 5) for k in range(64)] + [63, 64, 65, 0, 1, 2, 300],
         "unequal": [4000, 1, 0, 17, 2000], "empty": [0, 0, 1]}


@pytest.mark.parametrize("kind", ["mono", "rmu", "sp"])
@pytest.mark.parametrize("name", sorted(SIZES))
def test_items(name, kind):
    rng = np.random.default_rng(5)
    lin, mu = np.linspace(0.0, 25.0, 8), np.linspace(0.0, 1.0, 7)
    bn, ob = {"mono": (cute.Binning(cute.BIN_MONO, lin), oracle.Binning(oracle.MONO, lin)),
              "rmu": (cute.Binning(cute.BIN_RMU, lin, mu), oracle.Binning(oracle.RMU, lin, mu)),
              "sp": (cute.Binning(cute.BIN_SIGMAPI, lin, lin, los=cute.LOS_MIDPOINT),
                     oracle.Binning(oracle.SIGMAPI, lin, lin, los=oracle.LOS_MID))}[kind]
    cats = [rng.uniform(0.0, 100.0, (n, 3)) + 300.0 for n in SIZES[name]]
    grids = [cute.build_grid(c, cute.GEOM_BOX_OPEN, r_max=36.0) for c in cats]
    print("batch items", name, kind, flush=True)
    got = cute.count_pairs_batched([cute.BatchItem(g, None, bn) for g in grids])
    for c, h in zip(cats, got):
        np.testing.assert_array_equal(np.asarray(h).reshape(bn.shape), oracle.count_pairs(c, None, ob).reshape(bn.shape))
    # every catalog against the last one
    got = cute.count_pairs_batched([cute.BatchItem(g, grids[-1], bn) for g in grids[:-1]] or
                                   [cute.BatchItem(grids[0], None, bn)])
    for c, h in zip(cats[:-1], got):
        np.testing.assert_array_equal(np.asarray(h).reshape(bn.shape),
                                      oracle.count_pairs(c, cats[-1], ob).reshape(bn.shape))
