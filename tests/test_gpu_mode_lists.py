"""Mode sums over the wavenumbers that occur: one, several and many distinct
|k_y| (three to a group, nine to a pass over the nodes), scattered |k_x|, and
k_y beyond the lattice's rows, of which only the remainder modulo ny counts."""
import numpy as np
import pytest

from oracle import adjoint, collision, forcing, step
from paper_2412_08229_amd import Lattice, inputs
from paper_2412_08229_amd import _lib as L

pytestmark = pytest.mark.gpu

SHAPE, NY = (3, 40, 7), 40


def _oracle_force(ks, draw, amplitude, kf, c, u):
    """Force field of one step with the phases of k modulo the lattice's
    extents (exact where k.x in float64 is not)."""
    ext = np.array(u.shape[:0:-1])
    kr = (ks + ext // 2) % ext - ext // 2
    uh = forcing.velocity_modes(kr, u)
    fh = np.zeros((len(ks), 3), dtype=np.complex128)
    for m, k in enumerate(ks):
        e1, e2 = forcing.basis(k)
        phi, psi = np.pi * draw[m, 0], 2.0 * np.pi * draw[m, 1]
        th = forcing.phase_rule(np.sin(2 * phi), np.cos(2 * phi), psi, uh[m] @ e1, uh[m] @ e2)
        a, b = forcing.random_amplitudes(k, amplitude, kf, c, phi, psi, th)
        fh[m] = a * e1 + b * e2
    return forcing.field(kr, fh, u.shape[1:])


def _check(ks, amplitude, kf, c):
    """float64 storage, 3 steps: a mode's phase differs from the oracle's by
    at most ~1e-13, the force is below 1e-2."""
    ks = np.array(ks, dtype=np.int64)
    draws = inputs.uniform_draws(2, len(ks), 6)
    rho, u = inputs.random_velocity(SHAPE, seed=7, amp=0.05)
    with Lattice(SHAPE, "f64", "bgk", 0.6) as lat:
        lat.set_forcing(ks, draws, amplitude, kf, c, phase_rule=True)
        lat.init_equilibrium(rho, u)
        f = lat.populations()
        lat.step(3)
        got = lat.populations()
    op = step.Operator("bgk", 0.6)
    for t in range(3):
        _, ut = collision.macroscopic(f)
        f = step.step(f, op, force=_oracle_force(ks, draws[t % 2], amplitude, kf, c, ut))
    assert np.abs(got - f).max() < 1e-13


@pytest.mark.parametrize("kys", [[7], [0, 1, -1, 2], [0, 5, -11, 20], list(range(-4, 5)) + [9, -13, 20, 6],
                                 list(range(0, 20, 2)), list(range(-20, 21))])
def test_distinct_wavenumbers(kys):
    """1, 3, 4, 9, 10 and 21 distinct |k_y|, up to five distinct |k_x| with each."""
    kxs = [0, -1, 3, 16, 2, -9, 1]
    ks = [[kxs[i % 7], ky, 1 + i % 3] for i, ky in enumerate(kys)] + [[-2, ky, -1] for ky in kys]
    _check(ks, 1e-6, 1.5, 400.0)


@pytest.mark.parametrize("turns", [1, -1, 25000000])
def test_wavenumbers_beyond_the_rows(turns):
    """k_y = turns ny + r acts like r: at 1e9 rows' worth as well, where a sweep
    over every smaller wavenumber would not return."""
    base = turns * NY
    ks = [[kx, base + r, kz] for r in (0, 1, -1, 3, 20, -7) for kx, kz in ((0, 1), (-2, 1), (5, -2))]
    kk = float(abs(base))
    _check(ks, 1e-6 * kk ** 2, kk, kk ** 2)


@pytest.mark.parametrize("shape,kmax,count", [((3, 24, 5), (2, 12, 1), 40), ((2, 24, 260), (16, 3, 1), 30)])
def test_gradient_of_many_wavenumbers(shape, kmax, count):
    """Reverse mode with 13 distinct |k_y| (two passes) and with |k_x| up to
    16: the bound of the float32 adjoint (a few 1e-7 per step, summed)."""
    rng = np.random.Generator(np.random.PCG64(5))
    ks = rng.integers(-np.array(kmax), np.array(kmax) + 1, size=(count, 3))
    ks = ks[np.abs(ks).sum(axis=1) > 0]
    ks = np.concatenate([ks, [[1, y, 1] for y in range(kmax[1] + 1)]])
    draws = inputs.uniform_draws(2, len(ks), 8)
    rho, u = inputs.random_velocity(shape, seed=9, amp=0.05)
    params = inputs.mlp_params(32, 10)
    w = np.random.Generator(np.random.PCG64(11)).standard_normal((27,) + shape)
    with Lattice(shape, "f32", "nco", 0.58) as lat:
        lat.set_net_weights(params, 32, "tanh", "f32_mfma")
        lat.set_forcing(ks, draws, 1e-5, 1.5, 40.0, phase_rule=True)
        lat.init_equilibrium(rho, u)
        fs = lat.populations()
        lat.forward_record(3, 2)
        g, df0 = lat.backward(dL_df=w, want_df0=True)
    _, go, gfo = adjoint.run_and_grad(fs, 0.58, collision.unpack_params(params, 32), "tanh", 3,
                                      lambda x: (float((w * x).sum()), w), state_forcing=(ks, draws, 1e-5, 1.5, 40.0))
    go = adjoint.flatten(go)
    assert np.linalg.norm(g - go) < 1e-4 * np.linalg.norm(go)
    assert np.linalg.norm(df0 - gfo) < 1e-4 * np.linalg.norm(gfo)


@pytest.mark.parametrize("shape,kmax,count", [((300, 2, 3), (2, 2, 20), 40), ((600, 1, 1), (1, 1, 30), 30),
                                              ((70, 3, 5), (2, 1, 9), 40), ((3, 300, 2), (1, 12, 2), 40),
                                              ((512, 1, 600), (3, 0, 5), 12), ((1, 1 << 18, 1), (0, 9, 0), 9), ((900, 1, 300), (2, 0, 5), 6), ((520, 3, 1), (0, 1, 25), 30)])
def test_rows_along_either_axis(shape, kmax, count):
    """Short and thin planes: rows along z (300, 600, 70, 512, 520 long) or y,
    up to 256 to a block, with a remainder, in one group of wavenumbers and
    several; as _check, one step."""
    rng = np.random.Generator(np.random.PCG64(3))
    ks = rng.integers(-np.array(kmax), np.array(kmax) + 1, size=(count, 3))
    ks = ks[np.abs(ks).sum(axis=1) > 0]
    draws = inputs.uniform_draws(1, len(ks), 6)
    rho, u = inputs.random_velocity(shape, seed=7, amp=0.05)
    with Lattice(shape, "f64", "bgk", 0.6) as lat:
        lat.set_forcing(ks, draws, 1e-6, 1.5, 400.0, phase_rule=True)
        lat.init_equilibrium(rho, u)
        f = lat.populations()
        lat.step(1)
        got = lat.populations()
    _, ut = collision.macroscopic(f)
    want = step.step(f, step.Operator("bgk", 0.6), force=_oracle_force(ks, draws[0], 1e-6, 1.5, 400.0, ut))
    assert np.abs(got - want).max() < 1e-13


@pytest.mark.parametrize("shape", [(70, 3, 5), (5, 130, 2)])
def test_gradient_with_rows_along_either_axis(shape):
    """As test_gradient_of_many_wavenumbers."""
    rng = np.random.Generator(np.random.PCG64(5))
    ks = rng.integers([-2, -1, -2], [3, 2, 3], size=(30, 3))
    ks = ks[np.abs(ks).sum(axis=1) > 0]
    draws = inputs.uniform_draws(2, len(ks), 8)
    rho, u = inputs.random_velocity(shape, seed=9, amp=0.05)
    params = inputs.mlp_params(32, 10)
    w = np.random.Generator(np.random.PCG64(11)).standard_normal((27,) + shape)
    with Lattice(shape, "f32", "nco", 0.58) as lat:
        lat.set_net_weights(params, 32, "tanh", "f32_mfma")
        lat.set_forcing(ks, draws, 1e-5, 1.5, 40.0, phase_rule=True)
        lat.init_equilibrium(rho, u)
        fs = lat.populations()
        lat.forward_record(3, 2)
        g, df0 = lat.backward(dL_df=w, want_df0=True)
    _, go, gfo = adjoint.run_and_grad(fs, 0.58, collision.unpack_params(params, 32), "tanh", 3,
                                      lambda x: (float((w * x).sum()), w), state_forcing=(ks, draws, 1e-5, 1.5, 40.0))
    go = adjoint.flatten(go)
    assert np.linalg.norm(g - go) < 1e-4 * np.linalg.norm(go)
    assert np.linalg.norm(df0 - gfo) < 1e-4 * np.linalg.norm(gfo)


@pytest.mark.parametrize("shape", [(1 << 20, 1, 1), (1 << 18, 2, 2), (1, 1 << 20, 1), (1 << 14, 8, 8)])
def test_work_space_of_thin_lattices(shape):
    """The sums' work space: six doubles per mode and block of at least 256
    nodes, whatever the lattice's shape, beside the force field (3 floats per
    node); 64 MB for the coefficients and the allocator's granules."""
    torch = pytest.importorskip("torch")
    n, modes = int(np.prod(shape)), 60
    ks = np.array([[m % 5 - 2, m % 3 - 1, 1 + m] for m in range(modes)])
    with Lattice(shape, "f32", "bgk", 0.6) as lat:
        lat.sync()
        before = torch.cuda.mem_get_info()[0]
        lat.set_forcing(ks, inputs.uniform_draws(1, modes, 6), 1e-6, 1.5, 400.0, phase_rule=True)
        used = before - torch.cuda.mem_get_info()[0]
    assert used <= 12 * n + 48 * modes * n // 256 + (64 << 20)


@pytest.mark.parametrize("turns", [1, -1, 142857143, None])
def test_wavenumbers_beyond_the_planes(turns):
    """k_z = turns nz + r acts like r, down to the most negative integer, whose
    magnitude an int does not hold."""
    base = -2 ** 31 if turns is None else turns * SHAPE[0]
    ks = [[kx, ky, base + r] for r in (0, 1, 2) for kx, ky in ((0, 1), (-2, 3), (5, -2))]
    kk = float(abs(base))
    _check(ks, 1e-6 * kk ** 2, kk, kk ** 2)


@pytest.mark.parametrize("kx", [17, -17, -2 ** 31, 2 ** 31 - 1])
def test_large_kx_is_refused(kx):
    with Lattice((4, 4, 4), "f32", "bgk", 0.6) as lat:
        with pytest.raises(L.NCOError) as e:
            lat.set_forcing(np.array([[kx, 1, 0]]), inputs.uniform_draws(1, 1, 6), 1e-6, 1.5, 4.0, phase_rule=True)
        assert e.value.status == L.NCO_E_UNSUPPORTED
