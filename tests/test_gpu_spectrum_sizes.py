"""Energy spectrum where the two-factor transform changes form: one factor
(primes, up to the largest it serves), unequal factors, odd sizes, blocks with
few lines, the larger twiddle table, and the direct form beside it."""
import numpy as np
import pytest

from paper_2412_08229_amd import Lattice, inputs
from paper_2412_08229_amd.lattice import n_bins

pytestmark = pytest.mark.gpu


def _spectrum(u):
    n = u.shape[1]
    k = np.rint(np.fft.fftfreq(n, 1.0 / n))
    shell = np.floor(np.sqrt(k[:, None, None] ** 2 + k[None, :, None] ** 2 + k[None, None, :] ** 2) + 0.5).astype(int)
    e = sum(0.5 * np.abs(np.fft.fftn(u[c]) / n ** 3) ** 2 for c in range(3))
    return np.bincount(shell.ravel(), weights=e.ravel(), minlength=n_bins(n))[:n_bins(n)]


@pytest.mark.parametrize("n", [1, 2, 3, 5, 6, 15, 31, 34, 49, 67, 94, 96, 127, 130, 251, 257, 260])
def test_spectrum_matches_numpy(n):
    """float64 storage: each transform of n terms rounds to ~log2(n) or n ulp
    of its largest term, the state to a few; shells hold at least 1e-3 of the
    mean energy here."""
    rng = np.random.Generator(np.random.PCG64(n))
    u = 0.05 * (2.0 * rng.random((3, n, n, n)) - 1.0)
    with Lattice((n, n, n), "f64", "bgk", 0.6) as lat:
        lat.init_equilibrium(None, u)
        got = lat.energy_spectrum()
        again = lat.energy_spectrum()
    want = _spectrum(u)
    assert np.array_equal(got, again)
    assert np.abs(got - want).max() < 1e-12 * want.max() + 1e-18
    big = want > 1e-6 * want.max()
    assert np.abs(got[big] / want[big] - 1.0).max() < 1e-9


@pytest.mark.parametrize("n", [6, 31, 34, 67])
def test_spectrum_gradient_is_its_derivative(n):
    """dL/df0 of L = sum_k w_k E_k after one step against a central difference
    along its own direction (float64 storage; L is smooth and the step h
    ~1e-3 of the populations: truncation ~1e-6, float32 adjoint ~1e-6)."""
    rng = np.random.Generator(np.random.PCG64(n))
    shape = (n, n, n)
    rho, u = np.ones(shape), 0.05 * (2.0 * rng.random((3,) + shape) - 1.0)
    w = rng.standard_normal(n_bins(n))
    with Lattice(shape, "f32", "nco", 0.7) as lat:
        lat.set_net_weights(np.zeros(inputs.n_params(32)), 32, "tanh", "f32_mfma")
        lat.init_equilibrium(rho, u)
        f0 = lat.populations()
        lat.forward_record(1, 1)
        _, df0 = lat.backward(dL_dE=w, want_df0=True)
    d = df0 / np.sqrt((df0 ** 2).mean())
    h = 1e-4
    vals = []
    with Lattice(shape, "f64", "nco", 0.7) as lat:
        lat.set_net_weights(np.zeros(inputs.n_params(32)), 32, "tanh", "f32")
        for s in (h, -h):
            lat.init_populations(f0 + s * d)
            lat.step(1)
            vals.append(float(w @ lat.energy_spectrum()))
    fd = (vals[0] - vals[1]) / (2 * h)
    an = float((df0 * d).sum())
    assert abs(fd - an) < 1e-4 * abs(an)
