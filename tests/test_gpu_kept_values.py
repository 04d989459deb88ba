"""Network values kept for the reverse mode on lattices whose last block is partial."""
import numpy as np
import pytest

from paper_2412_08229_amd import Lattice, inputs

pytestmark = pytest.mark.gpu


def test_kept_values_past_the_last_node_do_not_enter_the_gradient():
    """420 nodes: the forward step's 16-node tiles write kept network values
    up to place 431, the 64-node blocks of the reverse step read up to 447.
    A 512-node lattice of NaN populations, whose kept values take the same
    memory and are freed, must leave no trace in a finite run's gradient."""
    shape = (3, 20, 7)
    params = inputs.mlp_params(32, 10)
    rho, u = inputs.random_velocity(shape, seed=9, amp=0.05)
    w = np.random.Generator(np.random.PCG64(11)).standard_normal((27,) + shape)
    grads = []
    for spoil in (False, True):
        with Lattice(shape, "f32", "nco", 0.58) as lat, Lattice((512, 1, 1), "f32", "nco", 0.58) as other:
            lat.set_net_weights(params, 32, "tanh", "f32_mfma")
            if spoil:
                # The same allocation size on a full 512-node lattice, left with NaN when freed.
                other.set_net_weights(params, 32, "tanh", "f32_mfma")
                other.init_populations(np.full((27, 512, 1, 1), np.nan))
                other.forward_record(3, 2)
                other.sync()
            other.close()
            lat.init_equilibrium(rho, u)
            lat.forward_record(3, 2)
            grads.append(lat.backward(dL_df=w)[0])
    assert np.all(np.isfinite(grads[0])) and np.array_equal(grads[0], grads[1])
