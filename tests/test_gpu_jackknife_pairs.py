"""Jackknife counts whose one region pass gives the total too (two counters in
one) and whose region tiles are cut on the device: exact against the oracle for
region labels in columns, at random and in one region, more regions than
points, and with the pair counters moved out many times in one count."""
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


LIN, MU = np.linspace(0.0, 24.0, 7), np.linspace(0.0, 1.0, 5)
KINDS = {"mono": (lambda m: m.Binning(m.BIN_MONO, LIN), lambda: oracle.Binning(oracle.MONO, LIN)),
         "rmu": (lambda m: m.Binning(m.BIN_RMU, LIN, MU), lambda: oracle.Binning(oracle.RMU, LIN, MU)),
         "mid": (lambda m: m.Binning(m.BIN_RMU, LIN, MU, los=m.LOS_MIDPOINT),
                 lambda: oracle.Binning(oracle.RMU, LIN, MU, los=oracle.LOS_MID))}
LABELS = {"columns": (9, lambda p, r: ((p[:, 0] - 200.0) // 30.1 * 3 + (p[:, 1] - 200.0) // 30.1).astype(np.int32)),
          "random": (5, lambda p, r: r.integers(0, 5, len(p)).astype(np.int32)),
          "sparse": (3000, lambda p, r: r.integers(0, 3000, len(p)).astype(np.int32)),
          "one": (4, lambda p, r: np.full(len(p), 2, np.int32))}


@pytest.mark.parametrize("flush", [None, "700"])
@pytest.mark.parametrize("labels", sorted(LABELS))
@pytest.mark.parametrize("kind", sorted(KINDS))
def test_regions(kind, labels, flush, monkeypatch):
    if flush:
        monkeypatch.setenv("CUTE_TEST_H32_FLUSH", flush)
    rng = np.random.default_rng(11)
    a, b = (rng.uniform(0.0, 90.0, (n, 3)) + 200.0 for n in (611, 450))
    a[:200] = a[200:400] + rng.normal(scale=0.5, size=(200, 3))   # dense cells
    a = np.clip(a, 200.0, 290.0)
    K, f = LABELS[labels]
    bn, ob = KINDS[kind][0](cute), KINDS[kind][1]()
    la, lb = f(a, rng), f(b, rng)
    ga, gb = (cute.build_grid(p, cute.GEOM_BOX_OPEN, r_max=24.0) for p in (a, b))
    ks = range(K) if K < 10 else [0, 1, int(la[0]), K - 1]
    for prec in (cute.PREC_FP32_EDGE, cute.PREC_FP64):
        print("jackknife pairs", kind, labels, flush, prec, flush=True)
        total, jack = cute.count_jackknife(ga, la, K, bn, prec)
        np.testing.assert_array_equal(np.ravel(total), np.ravel(oracle.count_pairs(a, None, ob)))
        for k in ks:
            np.testing.assert_array_equal(np.ravel(jack[k]), np.ravel(oracle.count_pairs(a[la != k], None, ob)))
        total, jack = cute.count_jackknife_cross(ga, la, gb, lb, K, bn, prec)
        np.testing.assert_array_equal(np.ravel(total), np.ravel(oracle.count_pairs(a, b, ob)))
        for k in ks:
            np.testing.assert_array_equal(np.ravel(jack[k]),
                                          np.ravel(oracle.count_pairs(a[la != k], b[lb != k], ob)))


def test_bad_labels_are_refused():
    p = np.random.default_rng(1).uniform(0.0, 90.0, (100, 3))
    g = cute.build_grid(p, cute.GEOM_BOX_OPEN, r_max=24.0)
    bn = KINDS["rmu"][0](cute)
    for v in (-1, 5, 70000):
        r = np.zeros(100, np.int32)
        r[37] = v
        with pytest.raises(cute.CuteError):
            cute.count_jackknife(g, r, 5, bn)
