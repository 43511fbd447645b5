"""Home tiles counted in parts: a count with few tiles cuts the neighbours of
every tile into runs of whole chunks, one task each. The counts must not
depend on the cut: exact against the oracle, and with the statistics of the
uncut walk (every candidate pair evaluated once, every tile reported once)."""
import numpy as np
import pytest

import catalogs
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


def cap(n, seed):
    return catalogs.cap_uniform(n, 25.0, 2.0, 10.0, seed)   # across phi = 0


@pytest.mark.parametrize("precision", [cute.PREC_FP64, cute.PREC_FP32_EDGE])
@pytest.mark.parametrize("n", [65, 500, 2047, 4096])
@pytest.mark.parametrize("kind", ["periodic", "open", "open_cross", "sphere", "sphere_cross"])
def test_parts_against_the_oracle(kind, n, precision):
    # cells so coarse that a tile meets many chunks of neighbours (up to 32
    # parts), tiles of 64, 7 and 1 points
    other = 2 * n + 3
    b = None
    if kind.startswith("sphere"):
        a, e = cap(n, 71), np.deg2rad(np.linspace(0.0, 20.0, 12))
        bn, ob = cute.Binning(cute.BIN_THETA, e), oracle.Binning(oracle.THETA, e)
        geom, L, cell, r = cute.GEOM_SPHERE, 0.0, 0.12, float(e[-1])
        if kind == "sphere_cross":
            b = cap(other, 72)
    else:
        per = kind == "periodic"
        a, e, L = catalogs.uniform_box(n, 100.0, seed=73), np.linspace(0.0, 30.0, 9), 100.0 if per else 0.0
        bn, ob = cute.Binning(cute.BIN_MONO, e), oracle.Binning(oracle.MONO, e, periodic=per, L=L)
        geom, cell, r = cute.GEOM_BOX_PERIODIC if per else cute.GEOM_BOX_OPEN, 12.0, 30.0
        if kind == "open_cross":
            b = catalogs.uniform_box(other, 90.0, seed=74)
    want = oracle.count_pairs(a, b, ob)
    gb = None if b is None else cute.build_grid(b, geom, box_size=L, r_max=r, cell_size=cell)
    for tile in (64, 7, 1):
        print("parts %s n %d prec %d tile %d" % (kind, n, precision, tile), flush=True)
        ga = cute.build_grid(a, geom, box_size=L, r_max=r, cell_size=cell, tile_points=tile)
        got, st = cute.count_pairs(ga, gb, bn, precision, with_stats=True)
        np.testing.assert_array_equal(got, want)
        assert st["pairs_in_range"] == int(want.sum()) <= st["pair_evals"]
        if b is None:
            assert st["pair_evals"] <= n * (n - 1) // 2
        else:
            assert st["pair_evals"] <= n * other
