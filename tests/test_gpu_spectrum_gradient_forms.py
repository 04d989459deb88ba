"""Reverse mode of the energy spectrum in the transforms' forms that smaller
sizes do not reach: the direct one (primes above 256) and the two-factor one
with the larger twiddle table (above 256)."""
import numpy as np
import pytest

from paper_2412_08229_amd import Lattice, inputs
from paper_2412_08229_amd.lattice import n_bins

pytestmark = pytest.mark.gpu

C = [(cx, cy, cz) for cz in (-1, 0, 1) for cy in (-1, 0, 1) for cx in (-1, 0, 1)]


@pytest.mark.parametrize("n", [257, 260])
def test_spectrum_gradient_through_one_step(n):
    """A collision keeps rho and j, and a dL/dx that depends on them alone
    passes its adjoint unchanged: dL/df0 after one step is the streaming's
    adjoint of the spectrum's, here from torch's float64 transforms.  Both
    round to float32 (6e-8 of each value), the collision's adjoint to a few
    1e-7 of the largest: the bound of the smaller sizes' test."""
    torch = pytest.importorskip("torch")
    rng = np.random.Generator(np.random.PCG64(n))
    w = rng.standard_normal(n_bins(n))
    u0 = 0.05 * (2.0 * rng.random((3, n, n, n)) - 1.0)
    with Lattice((n, n, n), "f32", "nco", 0.56) as lat:
        lat.set_net_weights(inputs.mlp_params(32, 9), 32, "tanh", "f32_mfma")
        lat.init_equilibrium(None, u0)
        lat.forward_record(1, 1)
        rho, u = lat.macroscopic()
        _, df0 = lat.backward(dL_dE=w, want_df0=True)
    rho, u = torch.from_numpy(rho).cuda(), torch.from_numpy(u).cuda()
    k = torch.round(torch.fft.fftfreq(n, 1.0 / n, dtype=torch.float64, device="cuda"))
    shell = torch.floor(torch.sqrt(k[:, None, None] ** 2 + k[None, :, None] ** 2 + k[None, None, :] ** 2) + 0.5).long()
    wk = torch.from_numpy(w).cuda()[shell] / float(n) ** 6
    # E = 1/2 sum |u_hat / n^3|^2 per shell, so dL/du = Re sum_k w u_hat e^{i k.x} / n^6.
    lu = torch.stack([torch.fft.ifftn(torch.fft.fftn(u[c]) * wk).real * float(n) ** 3 for c in range(3)])
    lr = -(lu * u).sum(dim=0) / rho
    err = norm = 0.0
    for i, (cx, cy, cz) in enumerate(C):
        lam = lr + (cx * lu[0] + cy * lu[1] + cz * lu[2]) / rho
        want = torch.roll(lam, shifts=(-cz, -cy, -cx), dims=(0, 1, 2))
        err += float(((torch.from_numpy(df0[i]).cuda() - want) ** 2).sum())
        norm += float((want ** 2).sum())
    assert err ** 0.5 < 2e-5 * norm ** 0.5
