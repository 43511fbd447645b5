"""FP32_EDGE counts with separations from the matrix cores: exact against the
oracle where the home points fill a step, sixteen rows or a tile unevenly, where
most pairs are ambiguous (the list of a step fills up), near the observer, and
at lengths that the FP32 path leaves to the FP64 one."""
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


def binnings(kind, s):
    """(binning, oracle binning, geometry, reach) at length scale s."""
    lin, mu = np.linspace(0.0, 30.0, 11) * s, np.linspace(0.0, 1.0, 9)
    log = np.geomspace(0.3, 30.0, 14) * s
    up = np.linspace(6.0, 30.0, 9) * s
    e1, e2, k, los = {
        "mono": (lin, None, "MONO", 0), "mono_log": (log, None, "MONO", 0), "mono_up": (up, None, "MONO", 0),
        "rmu": (lin, mu, "RMU", 0), "rmu_log": (log, mu, "RMU", 0),
        "rmu_generic": (up, np.array([0.1, 0.3, 0.8, 0.95]), "RMU", 0),
        "mid": (lin, mu, "RMU", 1), "mid_log": (log, mu, "RMU", 1), "mid_generic": (up, mu ** 2, "RMU", 1),
        "sp": (lin, lin * 0.7, "SIGMAPI", 1), "sp_up": (up, lin * 0.8 + 3.0 * s, "SIGMAPI", 1)}[kind]
    bn = cute.Binning(getattr(cute, "BIN_" + k), e1, e2, los=cute.LOS_MIDPOINT if los else cute.LOS_Z)
    ob = oracle.Binning(getattr(oracle, k), e1, e2, los=oracle.LOS_MID if los else oracle.LOS_Z)
    reach = float(np.hypot(e1[-1], e2[-1])) if k == "SIGMAPI" else float(e1[-1])
    return bn, ob, reach * (1 + 1e-12)


KINDS = ["mono", "mono_log", "mono_up", "rmu", "rmu_log", "rmu_generic", "mid", "mid_log", "mid_generic", "sp", "sp_up"]


def check(name, a, b, kind, s=1.0, tiles=(0,), cell=0.0):
    bn, ob, reach = binnings(kind, s)
    want = oracle.count_pairs(a, b, ob).reshape(bn.shape)
    assert want.sum() > 0
    gb = None if b is None else cute.build_grid(b, cute.GEOM_BOX_OPEN, r_max=reach, cell_size=cell)
    for t in tiles:
        print("mfma %s %s tile %d" % (name, kind, t), flush=True)
        ga = cute.build_grid(a, cute.GEOM_BOX_OPEN, r_max=reach, cell_size=cell, tile_points=t)
        np.testing.assert_array_equal(cute.count_pairs(ga, gb, bn, cute.PREC_FP32_EDGE), want, err_msg=name)
    return want


@pytest.mark.parametrize("kind", KINDS)
def test_tiles_of_every_remainder(kind):
    rng = np.random.default_rng(31)
    a = rng.uniform(0.0, 70.0, (700, 3)) + [900.0, -300.0, 1200.0]
    b = rng.uniform(5.0, 75.0, (900, 3)) + [900.0, -300.0, 1200.0]
    tiles = (64, 63, 33, 17, 16, 15, 5, 4, 3, 1)
    check("auto", a, None, kind, tiles=tiles, cell=25.0)
    check("cross", a, b, kind, tiles=tiles[::3], cell=25.0)


@pytest.mark.parametrize("kind", KINDS)
def test_most_pairs_ambiguous(kind):
    # a lattice whose separations sit on the edges, far from its grid's centre
    g = np.arange(9) * 3.0
    a = np.stack(np.meshgrid(g, g, g[:5], indexing="ij"), -1).reshape(-1, 3) + [4096.0, 2048.0, 1024.0]
    a = np.concatenate([a, a[:40], a[:3] - 900.0])   # duplicates, and a far corner that moves the centre
    check("lattice", a, None, kind, tiles=(64, 13))


@pytest.mark.parametrize("kind", ["mid", "mid_log", "sp", "sp_up"])
def test_observer_inside_the_catalog(kind):
    rng = np.random.default_rng(32)
    a = rng.uniform(-45.0, 45.0, (1300, 3))
    a[:2] = [[1.0, 2.0, 3.0], [-1.0, -2.0, -3.0]]    # p + q = 0
    check("around the observer", a, None, kind, tiles=(64, 7))


@pytest.mark.parametrize("kind", ["mono", "rmu", "mid", "sp"])
@pytest.mark.parametrize("scale", [1e-9, 1e-4, 1e5, 1e11])
def test_length_units(kind, scale):
    rng = np.random.default_rng(33)
    a = (rng.uniform(0.0, 60.0, (500, 3)) + [500.0, 400.0, 300.0]) * scale
    check("unit %g" % scale, a, None, kind, s=scale)


def test_histogram_that_leaves_no_room_for_the_stage():
    # one sigma bin and the most pi bins that the limit on histograms accepts:
    # beside them the staged home points do not fit, and the count runs in FP64
    rng = np.random.default_rng(34)
    a = rng.uniform(0.0, 50.0, (400, 3)) + 500.0
    e, lo, hi = np.array([0.0, 20.0]), 4000, 12000
    g = cute.build_grid(a, cute.GEOM_BOX_OPEN, r_max=29.0)

    def count(n2):
        bn = cute.Binning(cute.BIN_SIGMAPI, e, np.linspace(0.0, 20.0, n2 + 1), los=cute.LOS_MIDPOINT)
        return cute.count_pairs(g, None, bn, cute.PREC_FP32_EDGE, with_stats=True)

    while hi - lo > 1:   # lo is accepted, hi refused
        mid = (lo + hi) // 2
        try:
            count(mid)
            lo = mid
        except cute.CuteError as err:
            assert err.status == cute.E_UNSUPPORTED
            hi = mid
    got, st = count(lo)
    assert st["retests"] == 0 and count(lo - 40)[1]["retests"] > 0
    ob = oracle.Binning(oracle.SIGMAPI, e, np.linspace(0.0, 20.0, lo + 1), los=oracle.LOS_MID)
    np.testing.assert_array_equal(got, oracle.count_pairs(a, None, ob).reshape(got.shape))
