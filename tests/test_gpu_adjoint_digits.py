"""The digits of the matrix-core reverse step of depth-3 tanh networks."""
import numpy as np
import pytest

from oracle import adjoint, collision
from paper_2412_08229_amd import Lattice, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width", [20, 32])
@pytest.mark.parametrize("shape", [(5, 6, 7), (9, 30, 31)])
@pytest.mark.parametrize("mlp,cache", [("f32_mfma", None), ("f32_mfma", 0), ("f32_split", None)])
def test_gradient_of_small_activations(mlp, cache, shape, width):
    """First-layer weights and every hidden bias times 1e-4: activations of
    order 1e-4, so that a tanh right to its own last places gives each layer's
    gradient to float32's rounding (2e-5 of the layer's norm, the bound of the
    other gradient tests), where one right to 6e-8 absolutely is off by 6e-4 of
    an activation.  In tiles (210 nodes) and 64-node blocks (8370)."""
    params = inputs.mlp_params(width, 21, depth=3).astype(np.float32)
    sizes = [27 * width, width, width * width, width, width * width, width, 4 * width, 4]
    at = np.cumsum([0] + sizes)
    for k in (0, 1, 3, 5):
        params[at[k]:at[k + 1]] *= np.float32(1e-4)
    f0 = inputs.random_populations(shape, seed=22, lo=0.9, hi=1.1)
    w = np.random.Generator(np.random.PCG64(23)).standard_normal((27,) + shape)
    with Lattice(shape, "f32", "nco", 0.57) as lat:
        lat.set_net_weights(params, width, "tanh", mlp, depth=3)
        if cache is not None:
            lat.set_reverse_cache(cache)
        lat.init_populations(f0)
        fs = lat.populations()
        lat.forward_record(1, 1)
        g, df0 = lat.backward(dL_df=w, want_df0=True)
    layers = collision.unpack_params(params, width, depth=3)
    _, go, gfo = adjoint.run_and_grad(fs, 0.57, layers, "tanh", 1, lambda x: (float((w * x).sum()), w))
    go = adjoint.flatten(go)
    for a, b in zip(at[:-1], at[1:]):
        assert np.linalg.norm(g[a:b] - go[a:b]) < 2e-5 * np.linalg.norm(go[a:b])
    assert np.linalg.norm(df0 - gfo) < 2e-6 * np.linalg.norm(gfo)
