"""The reverse mode where device memory is too short for the network values it
would keep: the same gradient without them, no error."""
import numpy as np
import pytest

from paper_2412_08229_amd import Lattice, inputs

pytestmark = pytest.mark.gpu

N, WIDTH = 96, 20
STATE = 54 * N ** 3             # bytes of a BF16-deviation state
KEPT = 144 * N ** 3             # bytes of network values of one


def _fill(torch, spare, chunk=32 << 20):
    """Tensors that leave ``spare`` bytes of the device's memory: chunks up to
    the first refusal, then as many given back."""
    big = torch.cuda.mem_get_info()[0] - spare - (1 << 30)
    hold = [torch.empty(big, dtype=torch.uint8, device="cuda")]
    for _ in range(2000):
        try:
            hold.append(torch.empty(chunk, dtype=torch.uint8, device="cuda"))
        except torch.cuda.OutOfMemoryError:
            break
    del hold[len(hold) - -(-spare // chunk):]
    torch.cuda.empty_cache()
    return hold


def _run(T, K, cache, spare=None):
    """Gradient of a recorded run; with ``spare`` bytes of the device's memory
    left once the lattice stands."""
    torch = pytest.importorskip("torch")
    params = inputs.mlp_params(WIDTH, 21, depth=3)
    rho, u = inputs.random_velocity((N,) * 3, seed=3, amp=0.03)
    w = np.zeros((27,) + (N,) * 3)
    w[3, ::7, ::5, ::3] = 1.0
    hold = None
    with Lattice((N,) * 3, "bf16", "nco", 0.57) as lat:
        lat.set_net_weights(params, WIDTH, "relu", "f32_mfma", depth=3)
        lat.set_reverse_cache(cache)
        lat.init_equilibrium(rho, u)
        lat.sync()
        try:
            if spare is not None:
                hold = _fill(torch, spare)
            lat.forward_record(T, K)
            return lat.backward(dL_df=w)[0]
        finally:
            del hold
            torch.cuda.empty_cache()


# What a run needs besides its states: two adjoint states of 108 bytes per
# node, the 216 of the populations' host transfer, gradient rows; 300 MB over.
NEEDED = 2 * 108 * N ** 3 + 216 * N ** 3 + (300 << 20)


def test_recompute_values_that_do_not_fit():
    """40 steps in one segment: 39 states of values, 5 GB, of which less than
    half would fit beside everything else."""
    T = 40
    want = _run(T, T, 0)
    got = _run(T, T, 1 << 40, spare=NEEDED + (T + 1) * STATE + 15 * KEPT)
    assert np.all(np.isfinite(want)) and np.array_equal(got, want)


def test_kept_values_make_room():
    """30 steps with every state a checkpoint: the values of all of them fit
    while the run is recorded and leave 50 MB, less than the reverse mode
    needs."""
    T = 30
    want = _run(T, 1, 0)
    got = _run(T, 1, 1 << 40, spare=T * (STATE + KEPT) + (50 << 20))
    assert np.all(np.isfinite(want)) and np.array_equal(got, want)
