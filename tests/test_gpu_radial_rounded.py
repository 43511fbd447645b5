"""Radial counts of redshifts rounded to the bin width: most pairs lie on an
edge and would be re-tested, and waves that see it count in FP64. Exact against
brute force where waves take many tiles, and not much slower than the FP64
kernel that uneven edges take."""
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


def cap(n, rng):
    z, f = rng.uniform(0.0, 0.3, n), rng.uniform(0.0, 0.3, n)
    c = np.sqrt(1.0 - z * z)
    return np.stack([c * np.cos(f), c * np.sin(f), z], 1)


@pytest.mark.parametrize("step", [0.005, 0.0005, 0.0])
def test_exact(step):
    # tiles of one point: more tasks than waves, so that waves change over
    rng = np.random.default_rng(61)
    a, b = cap(14000, rng), cap(320, rng)
    za, zb = (0.5 + 0.1 * rng.uniform(size=len(p)) for p in (a, b))
    if step:
        za, zb = np.round(za / step) * step, np.round(zb / step) * step
    edges, ap = np.arange(21) * 0.005, 0.2
    print("rounded radial", step, flush=True)
    ga = cute.build_grid(a, cute.GEOM_SPHERE, r_max=ap, tile_points=1)
    gb = cute.build_grid(b, cute.GEOM_SPHERE, r_max=ap)
    d = a[:, None, :] - b[None, :, :]
    near = (d * d).sum(axis=2) < (2.0 * np.sin(0.5 * ap)) ** 2
    k = np.searchsorted(edges, np.abs(za[:, None] - zb[None, :])[near], side="right") - 1
    want = np.bincount(k[k < 20], minlength=20)
    np.testing.assert_array_equal(cute.count_radial(ga, za, gb, zb, ap, edges), want)


def test_time():
    rng = np.random.default_rng(62)
    a, b = cap(300000, rng), cap(300000, rng)
    za, zb = (np.round((0.5 + 0.1 * rng.uniform(size=len(p))) * 1e3) / 1e3 for p in (a, b))
    ap = np.deg2rad(1.0)
    ga, gb = (cute.build_grid(p, cute.GEOM_SPHERE, r_max=ap) for p in (a, b))
    edges = np.arange(101) * 0.001
    uneven = edges.copy()
    uneven[50] += 1e-5
    ms = [min(cute.count_radial(ga, za, gb, zb, ap, e, with_stats=True)[1]["ms_count"] for _ in range(4))
          for e in (edges, uneven)]
    print("rounded radial: %.2f ms, uneven edges %.2f ms" % tuple(ms), flush=True)
    assert ms[0] < 1.25 * ms[1]
