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


def _padded(params, width, depth):
    """The same network with hidden units of zero weights up to 32."""
    sizes = [27] + [width] * depth + [4]
    out, pos = [], 0
    for i, (a, b) in enumerate(zip(sizes[:-1], sizes[1:])):
        A, B = (a if i == 0 else 32), (b if i == depth else 32)
        w, v = np.zeros((A, B), np.float32), np.zeros(B, np.float32)
        w[:a, :b] = params[pos:pos + a * b].reshape(a, b)
        v[:b] = params[pos + a * b:pos + a * b + b]
        pos += a * b + b
        out += [w.ravel(), v]
    return np.concatenate(out)


def _step(shape, storage, width, depth, act, mlp, params, f):
    with Lattice(shape, storage, "nco", 0.53) as lat:
        lat.set_net_weights(params, width, act, mlp, depth=depth)
        lat.init_populations(f)
        r = lat.rates()
        lat.step(1)
        return r, lat.populations()


@pytest.mark.parametrize("mlp", ["f32", "f32_mfma"])
@pytest.mark.parametrize("width,depth,act", [(20, 2, "relu"), (20, 3, "tanh"), (8, 2, "tanh")])
@pytest.mark.parametrize("shape", [(1, 1, 1), (1, 17, 1), (17, 241, 1), (16, 64, 64), (32, 64, 64)])
def test_narrow_network_equals_its_padding(shape, width, depth, act, mlp):
    """Networks of at most 20 hidden units lie differently in the kernels'
    tiles; padded to 32 by hand they run the general form.  Adding exact zeros
    changes nothing in float32."""
    params = np.asarray(inputs.mlp_params(width, 41, depth=depth), np.float32)
    f = inputs.random_populations(shape, seed=42, lo=0.9, hi=1.1)
    r, p = _step(shape, "f32", width, depth, act, mlp, params, f)
    r32, p32 = _step(shape, "f32", 32, depth, act, mlp, _padded(params, width, depth), f)
    assert np.array_equal(r, r32) and np.array_equal(p, p32)


@pytest.mark.parametrize("mlp", ["bf16", "f32_split"])
@pytest.mark.parametrize("width,depth,act", [(20, 2, "relu"), (20, 3, "tanh"), (8, 2, "tanh")])
@pytest.mark.parametrize("shape", [(17, 241, 1), (16, 64, 64), (32, 64, 64)])
def test_narrow_16_bit_network_is_as_accurate_as_its_padding(shape, width, depth, act, mlp):
    """The 16-bit products add 32 terms at once, in an order of their own, and
    a hidden layer's activations round to 16 bits again, so the two forms
    differ by such roundings; their errors against float64, mostly those of
    the rounded weights and inputs, agree to a tenth in the mean square."""
    params = np.asarray(inputs.mlp_params(width, 41, depth=depth), np.float32)
    f = np.float32(inputs.random_populations(shape, seed=42, lo=0.9, hi=1.1)).astype(np.float64)
    r, p = _step(shape, "f32", width, depth, act, mlp, params, f)
    r32, p32 = _step(shape, "f32", 32, depth, act, mlp, _padded(params, width, depth), f)
    r64, p64 = _step(shape, "f64", width, depth, act, "f32", params, f)
    assert np.linalg.norm(r - r64) < 1.1 * np.linalg.norm(r32 - r64)
    assert np.linalg.norm(p - p64) < 1.1 * np.linalg.norm(p32 - p64)
