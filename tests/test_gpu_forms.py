"""FP32_EDGE counts whose separations are formed component by component: tile
frames as large as the separations, general r-mu edges, and lengths past the
range of the matrix cores. Exact against the oracle for single, cross, masked,
batched and jackknife counts, pixel maps, and radial counts in one cell."""
import numpy as np
import pytest

import oracle
import paper_1210_1833_amd as cute
from test_gpu_mfma import binnings

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible: the gpu tests need an MI355X")
    cute.load()
    yield


def path_of(geom, pts, bn, reach, cell):
    k, _, _ = cute.fp32_count_constants(geom, len(pts), pts.min(axis=0), pts.max(axis=0),
                                        float(np.linalg.norm(pts, axis=1).max()), bn, r_max=reach, cell_size=cell)
    return k["path"]


@pytest.mark.parametrize("kind", ["mono", "mono_log", "mono_up", "rmu", "rmu_log", "rmu_generic", "mid", "mid_log",
                                  "mid_generic", "sp", "sp_up"])
def test_boxes(kind):
    s = 2e6 if kind.startswith(("mid", "sp")) else 5e12
    bn, ob, reach = binnings(kind, s)
    rng = np.random.default_rng(51)
    a = (rng.uniform(0.0, 60.0, (700, 3)) + [300.0, -100.0, 250.0]) * s
    a = np.concatenate([a, a[:30]])
    b = (rng.uniform(5.0, 65.0, (500, 3)) + [300.0, -100.0, 250.0]) * s
    assert path_of(cute.GEOM_BOX_OPEN, a, bn, reach, 25.0 * s) == 1.0
    gb = cute.build_grid(b, cute.GEOM_BOX_OPEN, r_max=reach, cell_size=25.0 * s)
    mask = (rng.uniform(size=len(a)) < 0.3).astype(np.uint8)
    lab = rng.integers(0, 3, len(a)).astype(np.int32)
    want = oracle.count_pairs(a, None, ob).reshape(bn.shape)
    cross = oracle.count_pairs(a, b, ob).reshape(bn.shape)
    masked = oracle.count_pairs(a[mask == 0], None, ob).reshape(bn.shape)
    for tile in (64, 13):
        print("forms", kind, tile, flush=True)
        ga = cute.build_grid(a, cute.GEOM_BOX_OPEN, r_max=reach, cell_size=25.0 * s, tile_points=tile)
        np.testing.assert_array_equal(cute.count_pairs(ga, None, bn), want)
        np.testing.assert_array_equal(cute.count_pairs(ga, gb, bn), cross)
        got = cute.count_pairs_batched([cute.BatchItem(ga, None, bn, mask_a=mask), cute.BatchItem(ga, gb, bn)])
        np.testing.assert_array_equal(got[0], masked)
        np.testing.assert_array_equal(got[1], cross)
    total, jack = cute.count_jackknife(ga, lab, 3, bn)
    np.testing.assert_array_equal(total, want)
    for k in range(3):
        np.testing.assert_array_equal(jack[k], oracle.count_pairs(a[lab != k], None, ob).reshape(bn.shape))


def cap(n, seed):
    rng = np.random.default_rng(seed)
    z, f = rng.uniform(0.0, 0.3, n), rng.uniform(-0.2, 0.25, n)
    c = np.sqrt(1.0 - z * z)
    return np.stack([c * np.cos(f), c * np.sin(f), z], 1)


@pytest.mark.parametrize("log", [False, True])
def test_sphere_in_one_cell(log):
    a, b = cap(900, 3), cap(700, 4)
    a = np.concatenate([a, a[:20]])
    e = np.deg2rad(np.geomspace(0.5, 30.0, 300) if log else np.linspace(0.0, 30.0, 301))
    bn, ob = cute.Binning(cute.BIN_THETA, e), oracle.Binning(oracle.THETA, e)
    assert path_of(cute.GEOM_SPHERE, a, bn, float(e[-1]), 6.0) == 1.0
    print("forms sphere", log, flush=True)
    ga, gb = (cute.build_grid(p, cute.GEOM_SPHERE, r_max=float(e[-1]), cell_size=6.0) for p in (a, b))
    np.testing.assert_array_equal(cute.count_pairs(ga, None, bn), oracle.count_pairs(a, None, ob))
    np.testing.assert_array_equal(cute.count_pairs(ga, gb, bn), oracle.count_pairs(a, b, ob))
    # pixel maps: weighted pairs, as FP64 counts them
    ma, mb = (cute.build_pixel_map(p, 256, 512, r_max=float(e[-1]), cell_size=6.0) for p in (a, b))
    for other in (None, mb):
        np.testing.assert_array_equal(cute.count_pairs(ma, other, bn), cute.count_pairs(ma, other, bn, cute.PREC_FP64))


@pytest.mark.parametrize("aperture", [0.05, 1.0, 20.0])
def test_radial_in_one_cell(aperture):
    a, b = cap(900, 5), cap(700, 6)
    b[:200] = a[:200] + np.random.default_rng(2).normal(scale=3e-4, size=(200, 3))
    b /= np.linalg.norm(b, axis=1)[:, None]
    rng = np.random.default_rng(7)
    za, zb = rng.uniform(0.5, 0.6, len(a)), rng.uniform(0.5, 0.6, len(b))
    ap, edges = np.deg2rad(aperture), np.linspace(0.0, 0.1, 21)
    print("forms radial", aperture, flush=True)
    ga, gb = (cute.build_grid(p, cute.GEOM_SPHERE, r_max=ap, cell_size=6.0) for p in (a, b))
    d2 = ((a[:, None, :] - b[None, :, :]) ** 2).sum(axis=2)
    dz = np.abs(za[:, None] - zb[None, :])
    near = d2 < (2.0 * np.sin(0.5 * ap)) ** 2
    want = np.histogram(dz[near], edges)[0]
    want[-1] -= int(np.count_nonzero(dz[near] == edges[-1]))   # (half-open)
    np.testing.assert_array_equal(cute.count_radial(ga, za, gb, zb, ap, edges), want)


def test_one_cell_is_faster_than_fp64():
    # all pairs in range, 256 bins, a tile's frame of 2: with separations from the
    # matrix cores 3.5 % of the pairs were re-tested, 0.87 of the time of FP64
    # (component by component 0.63)
    a, b = cap(100000, 8), cap(100000, 9)
    e = np.deg2rad(np.linspace(0.0, 30.0, 257))
    bn = cute.Binning(cute.BIN_THETA, e)
    ga, gb = (cute.build_grid(p, cute.GEOM_SPHERE, r_max=float(e[-1]), cell_size=6.0) for p in (a, b))
    ms = {p: min(cute.count_pairs(ga, gb, bn, p, with_stats=True)[1]["ms_count"] for _ in range(4))
          for p in (cute.PREC_FP32_EDGE, cute.PREC_FP64)}
    print("one cell", ms, flush=True)
    assert ms[cute.PREC_FP32_EDGE] < 0.75 * ms[cute.PREC_FP64]
