"""FP32_EDGE counts of close pairs in small length units (kpc/h and below):
the expanded form of a separation then errs by more than the separation itself
and can be far below zero, and such a pair must be re-tested. Coincident points
and pairs at 1e-5 of a cell, with first edges at zero and inside their own
rounding band, exact against the oracle for single, batched and jackknife
counts."""
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


MU = np.linspace(0.0, 1.0, 6)


def binning(kind, s):
    lin = np.linspace(0.0, 60.0, 7) * s
    e = {"mono": lin, "mono_tiny": np.concatenate([[2e-5], lin[1:] / s]) * s, "mono_one": lin[::6],
         "mono_log": np.geomspace(1e-4, 60.0, 12) * s, "rmu": lin, "rmu_log": np.geomspace(1e-4, 60.0, 12) * s,
         "mid": lin}[kind]
    if kind.startswith("mono"):
        return cute.Binning(cute.BIN_MONO, e), oracle.Binning(oracle.MONO, e)
    mid = kind == "mid"
    return (cute.Binning(cute.BIN_RMU, e, MU, los=cute.LOS_MIDPOINT if mid else cute.LOS_Z),
            oracle.Binning(oracle.RMU, e, MU, los=oracle.LOS_MID if mid else oracle.LOS_Z))


def points(s):
    """600 points in cells of 50 s, a partner at a distance of about 1e-5 of
    a cell for 300 of them, and 300 coincident ones."""
    rng = np.random.default_rng(77)
    a = rng.uniform(0.0, 160.0, (600, 3)) + [300.0, 400.0, 500.0]
    p = np.concatenate([a, a[:300] + rng.normal(scale=3e-4, size=(300, 3)), a[300:]])
    return p[rng.permutation(len(p))] * s


@pytest.mark.parametrize("scale", [1.0, 1e3, 1e5])
@pytest.mark.parametrize("kind", ["mono", "mono_tiny", "mono_one", "mono_log", "rmu", "rmu_log", "mid"])
def test_counts(kind, scale):
    a = points(scale)
    bn, ob = binning(kind, scale)
    g = cute.build_grid(a, cute.GEOM_BOX_OPEN, r_max=60.0 * scale, cell_size=50.0 * scale)
    print("close pairs", kind, scale, flush=True)
    want = oracle.count_pairs(a, None, ob).reshape(bn.shape)
    np.testing.assert_array_equal(cute.count_pairs(g, None, bn, cute.PREC_FP32_EDGE), want)
    half = np.zeros(len(a), np.uint8)
    half[::2] = 1
    got = cute.count_pairs_batched([cute.BatchItem(g, None, bn), cute.BatchItem(g, None, bn, mask_a=half)])
    np.testing.assert_array_equal(got[0], want)
    np.testing.assert_array_equal(got[1], oracle.count_pairs(a[half == 0], None, ob).reshape(bn.shape))
    b = points(scale)[::-1] + 1e-4 * scale
    gb = cute.build_grid(b, cute.GEOM_BOX_OPEN, r_max=60.0 * scale, cell_size=50.0 * scale)
    np.testing.assert_array_equal(cute.count_pairs(g, gb, bn, cute.PREC_FP32_EDGE),
                                  oracle.count_pairs(a, b, ob).reshape(bn.shape))


@pytest.mark.parametrize("kind", ["mono", "rmu", "mid"])
def test_jackknife(kind):
    a = points(1e5)
    bn, ob = binning(kind, 1e5)
    g = cute.build_grid(a, cute.GEOM_BOX_OPEN, r_max=60e5, cell_size=50e5)
    lab = (np.arange(len(a)) % 3).astype(np.int32)
    print("close pairs jackknife", kind, flush=True)
    total, jack = cute.count_jackknife(g, lab, 3, bn, cute.PREC_FP32_EDGE)
    np.testing.assert_array_equal(total, oracle.count_pairs(a, None, ob).reshape(bn.shape))
    for k in range(3):
        np.testing.assert_array_equal(jack[k], oracle.count_pairs(a[lab != k], None, ob).reshape(bn.shape))


def test_periodic_box():
    s = 1e5
    rng = np.random.default_rng(78)
    a = rng.uniform(0.0, 400.0, (900, 3))
    p = np.mod(np.concatenate([a, a[:400] + rng.normal(scale=3e-4, size=(400, 3)), a[400:]]) * s, 400.0 * s)
    e = np.linspace(0.0, 60.0, 7) * s
    g = cute.build_grid(p, cute.GEOM_BOX_PERIODIC, box_size=400.0 * s, r_max=60.0 * s)
    print("close pairs periodic", flush=True)
    np.testing.assert_array_equal(cute.count_pairs(g, None, cute.Binning(cute.BIN_MONO, e), cute.PREC_FP32_EDGE),
                                  oracle.count_pairs(p, None, oracle.Binning(oracle.MONO, e, periodic=True, L=400.0 * s)))
