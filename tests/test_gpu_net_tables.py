"""Rates read under another operator: the network in full float32, whose table
is built when first read, after every change of the weights."""
import numpy as np
import pytest

from oracle import collision
from paper_2412_08229_amd import Lattice, inputs

pytestmark = pytest.mark.gpu

SHAPE = (3, 5, 7)
NETS = [(32, 2, "tanh", "f32_mfma"), (20, 2, "relu", "bf16"), (8, 2, "tanh", "f32_split"), (20, 3, "tanh", "f32_mfma"),
        (16, 2, "relu", "f32"), (32, 3, "relu", "f32_split"), (32, 2, "tanh", "f32")]


def test_rates_under_another_operator_follow_the_weights():
    """Widths, depths and arithmetics in turn on one lattice, each set of
    weights read twice, then replaced by another of the same form; the bound of
    the float32 network's rates (1e-6)."""
    f0 = inputs.random_populations(SHAPE, seed=3, lo=0.8, hi=1.2)
    with Lattice(SHAPE, "f32", "bgk", 0.6) as lat:
        lat.init_populations(f0)
        f = lat.populations()
        for width, depth, act, mlp in NETS + NETS[::-1]:
            for seed in (4, 5):
                params = inputs.mlp_params(width, seed, depth=depth)
                lat.set_net_weights(params, width, act, mlp, depth=depth)
                want = collision.nco_rates(f, collision.unpack_params(params, width, depth=depth), act)
                for _ in range(2):
                    assert np.abs(lat.rates() - want).max() < 1e-6


@pytest.mark.parametrize("width,depth,act,mlp", NETS)
def test_steps_and_gradient_after_other_weights(width, depth, act, mlp):
    """A step, and where there is a reverse mode a gradient, after other forms
    of network on the same lattice: those of a lattice of its own, bit for bit."""
    rho, u = inputs.random_velocity(SHAPE, seed=6, amp=0.05)
    w = np.random.Generator(np.random.PCG64(7)).standard_normal((27,) + SHAPE)

    def run(lat):
        lat.set_net_weights(inputs.mlp_params(width, 8, depth=depth), width, act, mlp, depth=depth)
        lat.init_equilibrium(rho, u)
        if width == 32 or depth == 3:
            lat.forward_record(2, 1)
            return [lat.populations()] + list(lat.backward(dL_df=w, want_df0=True))
        lat.step(2)
        return [lat.populations()]

    with Lattice(SHAPE, "f32", "nco", 0.6) as lat:
        for wo, do, ao, mo in NETS:
            lat.set_net_weights(inputs.mlp_params(wo, 9, depth=do), wo, ao, mo, depth=do)
        got = run(lat)
    with Lattice(SHAPE, "f32", "nco", 0.6) as lat:
        want = run(lat)
    assert all(np.array_equal(a, b) for a, b in zip(got, want))
