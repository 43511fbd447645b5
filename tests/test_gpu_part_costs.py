"""How home tiles are cut into parts: by the tiles' costs on the device. The
statistics of a cut count are those of the uncut walk, exactly; a mostly empty
bounding box and short tiles get the cut that they need (kernel times against
each other, with wide margins); and the tuner times counts cut as a user's are."""
import math

import numpy as np
import pytest

import paper_1210_1833_amd as cute

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible: the gpu tests need an MI355X")
    cute.load()
    yield


@pytest.mark.parametrize("precision", [cute.PREC_FP64, cute.PREC_FP32_EDGE, cute.PREC_FP32_ONLY])
@pytest.mark.parametrize("tile", [64, 13])
@pytest.mark.parametrize("n", [63, 1000, 4097, 20011])
def test_one_cell_statistics(n, tile, precision):
    # one cell: every pair is a candidate, and the tiles are the runs of a row.
    # Few tiles against all points, so every size but the first is cut.
    rng = np.random.default_rng(n)
    a, b = rng.uniform(0.0, 10.0, (n, 3)), rng.uniform(0.0, 10.0, (1777, 3))
    bn = cute.Binning(cute.BIN_MONO, np.linspace(0.0, 3.0, 5))
    ga = cute.build_grid(a, cute.GEOM_BOX_OPEN, r_max=3.0, cell_size=20.0, tile_points=tile)
    gb = cute.build_grid(b, cute.GEOM_BOX_OPEN, r_max=3.0, cell_size=20.0)
    print("one cell", n, tile, precision, flush=True)
    for other, pairs in ((None, n * (n - 1) // 2), (gb, n * 1777)):
        counts, st = cute.count_pairs(ga, other, bn, precision, with_stats=True)
        assert st["pair_evals"] == pairs
        assert st["tiles"] == -(-n // tile)
        assert st["pairs_in_range"] == int(counts.sum())
    m = np.zeros(n, np.uint8)
    _, st = cute.count_pairs_batched([cute.BatchItem(ga, None, bn, mask_a=m), cute.BatchItem(ga, gb, bn)],
                                     precision, with_stats=True)
    assert st["pair_evals"] == n * (n - 1) // 2 + n * 1777 and st["tiles"] == 2 * -(-n // tile)


def kernel_ms(points, bn, prec, reach, tile=0):
    g = cute.build_grid(points, cute.GEOM_BOX_OPEN, r_max=reach, tile_points=tile)
    runs = [cute.count_pairs(g, None, bn, prec, with_stats=True)[1] for _ in range(6)]
    return min(r["ms_count"] for r in runs), runs[0]["pair_evals"]


def cone(n, rng):
    ra, s = rng.uniform(0.0, math.radians(20.0), n), rng.uniform(0.0, math.sin(math.radians(20.0)), n)
    c = np.sqrt(1.0 - s * s)
    d = np.clip(rng.normal(1580.0, 345.0, n), 300.0, 3000.0)
    return np.stack([c * np.cos(ra), c * np.sin(ra), s], 1) * d[:, None]


def test_mostly_empty_bounding_box():
    # uncut, this count took 1.7 times as long as with tiles of 16 points
    bn = cute.Binning(cute.BIN_RMU, np.linspace(0.0, 100.0, 21), np.linspace(0.0, 1.0, 51), los=cute.LOS_MIDPOINT)
    p = cone(200000, np.random.default_rng(5))
    t64, t16 = kernel_ms(p, bn, cute.PREC_FP64, 100.0)[0], kernel_ms(p, bn, cute.PREC_FP64, 100.0, 16)[0]
    print("light cone, fp64 midpoint: %.2f ms, %.2f ms with tiles of 16" % (t64, t16), flush=True)
    assert t64 < 1.25 * t16


def test_short_tiles():
    # 15 points a tile: cut into four parts, the smaller catalog ran at 0.3 of
    # the larger one's rate (0.6 uncut)
    rng = np.random.default_rng(6)
    bn = cute.Binning(cute.BIN_RMU, np.linspace(0.0, 100.0, 21), np.linspace(0.0, 1.0, 51))

    def rate(n):
        blobs = rng.uniform(0.0, 1000.0, (n // 200, 1, 3)) + rng.normal(scale=5.0, size=(n // 200, 100, 3))
        p = np.concatenate([rng.uniform(0.0, 1000.0, (n // 2, 3)), blobs.reshape(-1, 3)])
        ms, evals = kernel_ms(np.mod(p, 1000.0), bn, cute.PREC_FP32_EDGE, 100.0)
        return evals / ms

    small, large = rate(300000), rate(600000)
    print("rates %.3g, %.3g evaluations a ms" % (small, large), flush=True)
    assert small > 0.45 * large


def test_tuner_counts_as_users_do():
    rng = np.random.default_rng(7)
    p = rng.uniform(0.0, 500.0, (20000, 3))
    bn = cute.Binning(cute.BIN_MONO, np.linspace(0.0, 100.0, 11))
    cells = [250.0, 100.0]
    _, _, ms = cute.tune_grid(p, cute.GEOM_BOX_OPEN, bn, r_max=100.0, cells=cells, tiles=[64])
    for cell in cells:
        t = ms[(cell, 64)]
        g = cute.build_grid(p, cute.GEOM_BOX_OPEN, r_max=100.0, cell_size=cell, tile_points=64)
        own = min(cute.count_pairs(g, None, bn, with_stats=True)[1]["ms_count"] for _ in range(6))
        print("cell %g: tuner %.3f ms, count %.3f ms" % (cell, t, own), flush=True)
        assert t < 1.6 * own
