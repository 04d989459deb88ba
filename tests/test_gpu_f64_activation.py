"""The float64 network's tanh beyond the ordinary range of its argument."""
import numpy as np
import pytest

from oracle import collision
from paper_2412_08229_amd import Lattice, inputs

pytestmark = pytest.mark.gpu


def _parts(params, width, depth):
    """Views of params: [W1, b1, W2, b2, (W2b, b2b,) W3, b3]."""
    sizes = [27 * width, width] + (depth - 1) * [width * width, width] + [4 * width, 4]
    at = np.cumsum([0] + sizes)
    return [params[a:b] for a, b in zip(at[:-1], at[1:])]


def _rates(params, width, depth):
    shape = (3, 5, 7)
    f0 = inputs.random_populations(shape, seed=5, lo=0.8, hi=1.2)
    with Lattice(shape, "f64", "nco", 0.6) as lat:
        lat.set_net_weights(params, width, "tanh", "f32", depth=depth)
        lat.init_populations(f0)
        got = lat.rates()
    return got, collision.nco_rates(f0, collision.unpack_params(params, width, depth=depth), "tanh")


@pytest.mark.parametrize("width,depth", [(8, 2), (20, 2), (32, 2), (20, 3), (32, 3)])
@pytest.mark.parametrize("scale", [1e-3, 1e-6, 1e-9])
def test_small_activations_keep_their_digits(scale, width, depth):
    """Hidden activations of order ``scale``, output weights of order 1 / scale:
    every product and tanh is right to a few roundings of its own size, so the
    rates are as close as with both of order one (the bound there: 1e-13).  A
    tanh right to 1e-16 absolutely would give 1e-16 / scale."""
    params = inputs.mlp_params(width, 6, depth=depth).astype(np.float32)
    p = _parts(params, width, depth)
    for b in [p[0]] + p[1:-1:2]:
        b *= np.float32(scale)
    p[-2] /= np.float32(scale)
    got, want = _rates(params, width, depth)
    assert np.abs(got - want).max() < 1e-13


@pytest.mark.parametrize("width,depth", [(8, 2), (20, 2), (32, 2), (32, 3)])
def test_infinite_and_huge_parameters_saturate(width, depth):
    """Infinite biases of either sign in every hidden layer, an infinite weight
    of the density row and weights whose pre-activations pass 2^31 and 2^1000
    of the exponent's unit: tanh is +-1, the rates those of the oracle."""
    params = inputs.mlp_params(width, 8, depth=depth).astype(np.float32)
    p = _parts(params, width, depth)
    for b in p[1:-1:2]:
        b[1], b[4] = np.inf, -np.inf
    p[0][2], p[0][5] = np.inf, -np.inf      # row 0 of W1: the density moment
    p[1][3], p[1][6], p[1][7] = 1e12, -3e38, 600.0
    got, want = _rates(params, width, depth)
    assert np.all(np.isfinite(want)) and np.abs(got - want).max() < 1e-13


@pytest.mark.parametrize("width,depth", [(8, 2), (32, 3)])
def test_nan_parameter_gives_nan(width, depth):
    params = inputs.mlp_params(width, 8, depth=depth).astype(np.float32)
    _parts(params, width, depth)[1][3] = np.nan
    got, want = _rates(params, width, depth)
    assert np.all(np.isnan(want)) and np.all(np.isnan(got))
