"""The float32 network where its kernels change form (twelve-wavefront tiles,
one-tile and four-tile wavefronts; half products up to 16 hidden units), against
the float64 network on the same populations."""
import numpy as np
import pytest

from paper_2412_08229_amd import Lattice, inputs

pytestmark = pytest.mark.gpu


def _run(shape, storage, op, width, depth, act, params, f):
    with Lattice(shape, storage, "nco", 0.53) as lat:
        lat.set_net_weights(params, width, act, "f32", depth=depth)
        lat.init_populations(f)
        lat.set_op(op)
        rates = lat.rates()
        lat.set_op("nco")
        lat.step(2)
        return rates, lat.populations()


@pytest.mark.parametrize("width,depth,act", [(8, 2, "tanh"), (16, 2, "relu"), (20, 2, "tanh"), (32, 3, "tanh"),
                                             (8, 3, "relu")])
@pytest.mark.parametrize("shape", [(1, 1, 1), (1, 17, 1), (16, 16, 16), (17, 241, 1), (15, 17, 257), (16, 64, 64)])
def test_network_matches_float64(shape, width, depth, act):
    """1, 17, 4096, 4097, 65535 and 65536 nodes.  A rate is a few float32
    operations on tilde tau, itself the mean of 48 outputs: 1e-6 is eight of
    its roundings; two steps of populations of order 0.3 at most, a few of
    theirs each.  The rates of another operator's lattice are the same."""
    params = inputs.mlp_params(width, 31, depth=depth)
    f = np.float32(inputs.random_populations(shape, seed=32, lo=0.9, hi=1.1)).astype(np.float64)
    r, p = _run(shape, "f32", "nco", width, depth, act, params, f)
    r64, p64 = _run(shape, "f64", "nco", width, depth, act, params, f)
    assert np.max(np.abs(r / r64 - 1.0)) < 1e-6
    assert np.max(np.abs(p - p64)) < 1e-6
    other, _ = _run(shape, "f32", "bgk", width, depth, act, params, f)
    assert np.array_equal(r, other)
