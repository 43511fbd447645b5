"""FP64 counts whose bins are guessed in FP32 and checked against the edges:
exact against the oracle where the guess holds (linear and log edges), where it
is mostly off (uneven edges), on lattices whose pairs lie on edges, along the
line of sight and at zero separation, and at lengths that FP32 cannot square."""
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


EDGES = {"linear": np.arange(0.0, 9.0), "above": np.arange(2.0, 9.0), "log": 2.0 ** np.arange(-1.0, 4.0),
         "uneven": np.array([0.0, 0.1, 0.2, 1.0, 1.5, 5.0, 5.001, 8.0]), "one": np.array([0.0, 8.0])}
MU = {"linear": np.linspace(0.0, 1.0, 6), "uneven": np.array([0.0, 0.02, 0.6, 0.99, 1.0]),
      "partial": np.array([0.25, 0.5, 0.75])}


def points(shape, scale):
    rng = np.random.default_rng(3)
    if shape == "lattice":
        p = np.stack(np.meshgrid(*[np.arange(7.0)] * 3), -1).reshape(-1, 3)
        p = np.concatenate([p, p[::5]])   # zero separations
    else:
        p = rng.uniform(0.0, 30.0, (901, 3))
    return p[rng.permutation(len(p))] * scale


@pytest.mark.parametrize("scale", [1.0, 2.0 ** -70, 2.0 ** 66])
@pytest.mark.parametrize("shape", ["lattice", "uniform"])
@pytest.mark.parametrize("e1", sorted(EDGES))
def test_boxes(e1, shape, scale):
    a = points(shape, scale)
    e = EDGES[e1] * scale
    g = cute.build_grid(a, cute.GEOM_BOX_OPEN, r_max=8.0 * scale)
    print("fp64 guess", e1, shape, scale, flush=True)
    np.testing.assert_array_equal(cute.count_pairs(g, None, cute.Binning(cute.BIN_MONO, e), cute.PREC_FP64),
                                  oracle.count_pairs(a, None, oracle.Binning(oracle.MONO, e)))
    for mu in MU.values():
        np.testing.assert_array_equal(
            cute.count_pairs(g, None, cute.Binning(cute.BIN_RMU, e, mu), cute.PREC_FP64).reshape(-1),
            oracle.count_pairs(a, None, oracle.Binning(oracle.RMU, e, mu)).reshape(-1))


@pytest.mark.parametrize("e1", ["linear", "log", "uneven"])
def test_sphere(e1):
    rng = np.random.default_rng(4)
    v = rng.normal(size=(900, 3)) * [0.2, 0.2, 0.0] + [0.0, 0.0, 1.0]
    v /= np.linalg.norm(v, axis=1)[:, None]
    v = np.concatenate([v, v[:50]])
    e = EDGES[e1] * 0.02
    g = cute.build_grid(v, cute.GEOM_SPHERE, r_max=float(e[-1]))
    print("fp64 guess sphere", e1, flush=True)
    np.testing.assert_array_equal(cute.count_pairs(g, None, cute.Binning(cute.BIN_THETA, e), cute.PREC_FP64),
                                  oracle.count_pairs(v, None, oracle.Binning(oracle.THETA, e)))
