"""The float64 network on the matrix cores (float64 storage): rates against
the oracle where a 16-node tile, a 64-node block or the width leaves a
remainder, at both depths, and with first-layer weights large enough to
saturate tanh on both sides of 2^1024."""
import numpy as np
import pytest

from oracle import collision
from paper_2412_08229_amd import Lattice, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("act", ["tanh", "relu"])
@pytest.mark.parametrize("width,depth", [(8, 2), (16, 2), (20, 2), (32, 2), (20, 3), (32, 3)])
@pytest.mark.parametrize("shape", [(1, 1, 1), (3, 1, 5), (1, 1, 17), (7, 3, 3), (5, 13, 1)])
def test_f64_rates_match_oracle_at_tile_edges(shape, width, depth, act):
    """1, 15, 17, 63 and 65 nodes.  Sums of at most 32 products and 48 terms
    of order one in float64: a few hundred roundings of 1.1e-16 at most."""
    f0 = inputs.random_populations(shape, seed=3, lo=0.8, hi=1.2)
    params = inputs.mlp_params(width, 4, depth=depth)
    with Lattice(shape, "f64", "nco", 0.6) as lat:
        lat.set_net_weights(params, width, act, "f32", depth=depth)
        lat.init_populations(f0)
        got = lat.rates()
    want = collision.nco_rates(f0, collision.unpack_params(params, width, depth=depth), act)
    assert np.abs(got - want).max() < 1e-13


@pytest.mark.parametrize("scale", [1e2, 1e4])
def test_f64_tanh_saturates(scale):
    """First-layer weights times ``scale``: pre-activations of ~10 scale, whose
    rounding (~1e-15 scale) passes tanh with slope at most 1 and the two
    layers of weights ~0.1 after it."""
    shape, width = (3, 5, 7), 32
    f0 = inputs.random_populations(shape, seed=5, lo=0.5, hi=1.5)
    params = inputs.mlp_params(width, 6)
    params[:27 * width] = (params[:27 * width] * scale).astype(np.float32)
    with Lattice(shape, "f64", "nco", 0.6) as lat:
        lat.set_net_weights(params, width, "tanh", "f32")
        lat.init_populations(f0)
        got = lat.rates()
    want = collision.nco_rates(f0, collision.unpack_params(params, width), "tanh")
    assert np.all(np.isfinite(got)) and np.abs(got - want).max() < 1e-14 * scale + 1e-13
