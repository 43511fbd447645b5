"""Radial counts whose redshift bins are decided in bin units (linear edges):
exact against the oracle for bins that start at and above zero, redshifts on
the edges, differences far past the last bin, and redshifts so large in bins
that FP32 decides no pair, or so large that no FP32 holds them."""
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


def cap(n, rng):
    v = rng.normal(size=(n, 3)) * [0.05, 0.05, 0.0] + [0.0, 0.0, 1.0]
    return v / np.linalg.norm(v, axis=1)[:, None]


CASES = {
    "plain": (np.linspace(0.0, 0.1, 101), lambda r, n: r.uniform(0.4, 0.7, n)),
    "above_zero": (np.linspace(0.03, 0.1, 8), lambda r, n: r.uniform(0.4, 0.7, n)),
    "one_bin": (np.array([0.0, 0.05]), lambda r, n: r.uniform(0.4, 0.7, n)),
    "on_edges": (np.linspace(0.0, 2.0, 17), lambda r, n: r.integers(0, 40, n) / 8.0),
    "far": (np.linspace(0.0, 1.0, 11), lambda r, n: r.uniform(0.0, 2.0, n) * 10.0 ** r.integers(0, 9, n)),
    "undecided": (np.linspace(0.0, 64.0, 65), lambda r, n: 2.0 ** 27 + r.integers(0, 100, n)),
    "no_float": (np.linspace(0.0, 1e299, 11), lambda r, n: r.uniform(0.0, 1e300, n) * r.choice([1.0, 1e-200], n)),
    "tiny": (np.linspace(0.0, 1e-290, 11), lambda r, n: r.uniform(0.0, 1e-289, n)),
    "many": (np.linspace(0.0, 0.3, 3001), lambda r, n: r.uniform(0.4, 0.7, n)),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_linear_bins(name):
    edges, draw = CASES[name]
    rng = np.random.default_rng(7)
    a, b = cap(700, rng), cap(901, rng)
    za, zb = draw(rng, 700), draw(rng, 901)
    for ap in (0.02, 0.3):
        ga, gb = (cute.build_grid(v, cute.GEOM_SPHERE, r_max=ap) for v in (a, b))
        print("radial bins", name, ap, flush=True)
        want = oracle.count_radial(a, za, b, zb, ap, edges)
        assert want.sum() > 0
        np.testing.assert_array_equal(cute.count_radial(ga, za, gb, zb, ap, edges), want)
        np.testing.assert_array_equal(cute.count_radial(ga, za, None, None, ap, edges),
                                      oracle.count_radial(a, za, None, None, ap, edges))
