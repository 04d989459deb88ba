"""Timed cases of the lattice Boltzmann engine: the work its users have it do.

Each case is a dict of plain values; ``kind`` selects one of six programs:

* ``interval``: a solve advanced by some steps between two looks at it (a
  Taylor-Green curve sampled every few steps, a decaying box), any operator,
  storage, network arithmetic, domain and extent;
* ``forced``: steps of a box driven by Alvelius forcing, drawn phases or the
  velocity-dependent ones (the run that stands in for the DNS);
* ``snapshot``: the readout of a fine run for training: energy spectrum,
  restriction to a coarse lattice, the coarse populations on the host;
* ``serve``: one round of the solve server over its resident lattices;
* ``dissipation``: loss and gradient of the dissipation-rate training;
* ``spectrum``: loss and gradient of the forced-turbulence training.

``exact`` is the same mathematics in float64 torch, written from the paper's
definitions: dense Hermite matrix, 48 group matrices, autograd.
"""
import itertools
import math

import numpy as np
import torch

from paper_2412_08229_amd import Lattice, inputs
from paper_2412_08229_amd.lattice import batch_step, n_bins
from paper_2412_08229_amd.training import DissipationUnroll, Unroll, make_autograd

U0 = 0.1 / math.sqrt(3.0)                           # Ma = 0.1
SIZE = {"f32": 4, "f16": 2, "bf16": 2, "f64": 8}


# ------------------------------------------------------------------ cases --

def listed():
    return [
        # The smallest call: one sampling interval of the dissipation curve on
        # the 10^3 reduced cube with the network of that training
        # (27-20-20-20-4 ReLU), kinetic energy read after it.
        dict(name="cube10_interval", kind="interval", nx=10, ny=10, nz=10, domain="tgv_octant", op="nco",
             storage="f32", mlp="f32_mfma", width=20, depth=3, act="relu", tau=0.56, steps=17),
        # The same training's loss and gradient on the 16^3 cube: samples
        # every 26 steps, checkpoints every 50.
        dict(name="cube16_train_depth3", kind="dissipation", n=16, domain="tgv_octant", width=20, depth=3,
             act="relu", mlp="f32_mfma", tau=0.5176, every=26, samples=4, ckpt=50),
        # Dissipation training on the periodic 32^3 vortex, 27-32-32-4 tanh.
        dict(name="tgv32_train", kind="dissipation", n=32, domain="periodic", width=32, depth=2, act="tanh",
             mlp="f32_mfma", tau=0.505, every=9, samples=5, ckpt=20),
        # Forced-turbulence training at its full grid, gradient through the
        # velocity-dependent phase, part of the 200-step unroll.
        dict(name="turb64_train", kind="spectrum", n=64, width=32, act="tanh", mlp="f32_mfma", tau=0.52, steps=40,
             ckpt=20, kmin=2, kmax=16, kforce=2.5, phase=True),
        # The benchmark's own step: 128^3, float32 throughout.
        dict(name="nco128_f32", kind="interval", nx=128, ny=128, nz=128, domain="periodic", op="nco", storage="f32",
             mlp="f32_mfma", width=32, depth=2, act="tanh", tau=0.5022, steps=2),
        # The paper's 27-20-20-4 ReLU network on the bf16 matrix cores, ragged box.
        dict(name="nco_paper_bf16_ragged", kind="interval", nx=101, ny=97, nz=89, domain="periodic", op="nco",
             storage="f32", mlp="bf16", width=20, depth=2, act="relu", tau=0.51, steps=4),
        # Float32-class split products with FP16-deviation storage, 27-32-32-4 tanh.
        dict(name="nco96_split_f16", kind="interval", nx=96, ny=96, nz=96, domain="periodic", op="nco",
             storage="f16", mlp="f32_split", width=32, depth=2, act="tanh", tau=0.505, steps=4),
        # The float64 reference run (the only network arithmetic float64
        # storage has, and what a program gets that names none).
        dict(name="nco40_f64", kind="interval", nx=40, ny=40, nz=40, domain="periodic", op="nco", storage="f64",
             mlp="f32", width=32, depth=2, act="tanh", tau=0.505, steps=2),
        # BGK on the benchmark lattice (in place on one cache-resident buffer).
        dict(name="bgk128_f32", kind="interval", nx=128, ny=128, nz=128, domain="periodic", op="bgk", storage="f32",
             mlp="", width=0, depth=0, act="", tau=0.5022, steps=20),
        # The forced fine run of the spectrum training: 256^3 BGK, |k| <= 2,
        # velocity-dependent phase.
        dict(name="dns256_forced", kind="forced", nx=256, ny=256, nz=256, op="bgk", storage="f32", tau=0.6, steps=2,
             kforce=2.0, phase=True),
        # What each snapshot of that run is turned into.
        dict(name="snapshot256", kind="snapshot", n=256, ratio=8, storage="f32", tau=0.6),
        # A round of the solve server: float32 and BF16 class solves on three grids.
        dict(name="serve_round", kind="serve", grids="32,64,96", steps=50),
    ]


def draw(rng):
    """One more case of the same ranges."""
    def near(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    tau = round(rng.uniform(0.505, 0.6), 4)
    kind = rng.choice(["interval", "interval", "interval", "forced", "snapshot", "serve", "dissipation", "dissipation",
                       "spectrum"])
    if kind == "interval":
        op = rng.choice(["nco", "nco", "nco", "nco", "bgk", "mrt"])
        octant = rng.random() < 0.25
        storage = rng.choice(["f32", "f32", "f32", "f16", "bf16", "f64"])
        case = dict(kind=kind, domain="tgv_octant" if octant else "periodic", op=op, storage=storage, mlp="", width=0,
                    depth=0, act="", tau=tau)
        if op == "nco":
            mlp = "f32" if storage == "f64" else rng.choice(["f32_mfma", "f32_mfma", "bf16", "f32_split", "f32"])
            width, depth = rng.choice([(32, 2), (32, 2), (20, 2), (20, 3)])
            case.update(mlp=mlp, width=width, depth=depth, act=rng.choice(["tanh", "relu"]))
            hi = 40 if mlp == "f32" else 128
        else:
            hi = 128 if storage == "f64" else 224
        if octant:
            n = near(8, min(hi, 32))
            case.update(nx=n, ny=n, nz=n)
        else:
            case.update(nx=near(8, hi), ny=near(8, hi), nz=near(8, hi))
        return dict(case, steps=rng.randint(1, 6 if case["mlp"] == "f32" else 20))
    if kind == "forced":
        return dict(kind=kind, nx=near(24, 256), ny=near(24, 256), nz=near(24, 256), op=rng.choice(["bgk", "mrt"]),
                    storage="f32", tau=tau, steps=rng.randint(1, 4), kforce=rng.choice([1.5, 2.0, 2.5]),
                    phase=rng.random() < 0.7)
    if kind == "snapshot":
        ratio = rng.choice([2, 3, 4, 8])
        return dict(kind=kind, n=ratio * rng.randint(max(2, 24 // ratio), 240 // ratio), ratio=ratio,
                    storage=rng.choice(["f32", "f32", "f64", "f16"]), tau=tau)
    if kind == "serve":
        grids = [rng.choice([32, 40, 48, 64]) for _ in range(rng.randint(2, 4))]
        return dict(kind=kind, grids=",".join(map(str, grids)), steps=rng.randint(5, 50))
    if kind == "dissipation":
        octant, depth = rng.random() < 0.7, rng.choice([2, 3])
        return dict(kind=kind, n=near(10, 32), domain="tgv_octant" if octant else "periodic",
                    width=32 if depth == 2 else rng.choice([20, 32]), depth=depth, act=rng.choice(["tanh", "relu"]),
                    mlp="f32_mfma", tau=tau, every=rng.randint(5, 15), samples=rng.randint(4, 6),
                    ckpt=rng.randint(10, 50))
    return dict(kind=kind, n=near(16, 64), width=32, act="tanh", mlp=rng.choice(["f32_mfma", "f32_mfma", "f32_split"]),
                tau=tau, steps=rng.randint(10, 40), ckpt=rng.randint(5, 20), kmin=2, kmax=6,
                kforce=rng.choice([2.0, 2.5]), phase=rng.random() < 0.5)


# ----------------------------------------------------------------- inputs --

def _flow(shape, seed, urms):
    """Random-phase solenoidal velocity, E(k) ~ k^4 exp(-2 (k / 4)^2), of rms
    urms per component, and its density (1 + small pressure noise): (rho, u)
    as float64 tensors on the GPU."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    ks = [torch.fft.fftfreq(n, 1.0 / n, dtype=torch.float64, device="cuda") for n in shape]
    kz, ky, kx = torch.meshgrid(*ks, indexing="ij")
    k = torch.stack([kx, ky, kz])
    kk = k.square().sum(0)
    k2 = kk.clamp(min=1.0)
    noise = torch.randn((3,) + tuple(shape), generator=gen, dtype=torch.float64, device="cuda")
    uh = torch.fft.fftn(noise, dim=(1, 2, 3)) * (k2.sqrt() * torch.exp(-kk / 16.0) * (kk > 0))
    uh -= k * ((k * uh).sum(0) / k2)
    u = torch.fft.ifftn(uh, dim=(1, 2, 3)).real
    u *= urms / u.square().mean().sqrt()
    rho = 1.0 + 1e-3 * torch.randn(tuple(shape), generator=gen, dtype=torch.float64, device="cuda")
    return rho, u


def _vortex(n, seed):
    """The reduced-cube Taylor-Green start at a velocity drawn around Ma 0.1."""
    u0 = U0 * (0.8 + 0.4 * np.random.Generator(np.random.PCG64(seed)).random())
    return inputs.tgv3d_octant(n, u0) + (u0,)


def _start(case, seed):
    """(rho, u) on the host of an interval or dissipation case."""
    if case["domain"] == "tgv_octant":
        rho, u, _ = _vortex(case.get("n") or case["nx"], seed)
        return rho, u
    shape = (case["n"],) * 3 if "n" in case else (case["nz"], case["ny"], case["nx"])
    rho, u = _flow(shape, seed, 0.03)
    return rho.cpu().numpy(), u.cpu().numpy()


def _params(case, seed):
    return inputs.mlp_params(case["width"], seed, case.get("depth", 2))


def _modes(case, seed, n_steps):
    ks = inputs.forcing_half_modes(case["kforce"])
    return ks, inputs.uniform_draws(n_steps, len(ks), seed + 7)


FORCE = (1e-6, 1.5, 1.0)                            # amplitude, k_f, c
DRAW_STEPS = 64


def _training_start(case, seed):
    """Populations of a training sample: one BGK step after an equilibrium,
    rounded to the float32 the lattice holds."""
    rho, u = _flow((case["n"],) * 3, seed, 0.05)
    f = _Model().step(_Model.equilibrium(rho, u), "bgk", case["tau"])
    return f.float().double()


def _target_spectrum(case):
    k = np.arange(n_bins(case["n"]), dtype=np.float64)
    return 1e-5 * (k + 0.5) ** 4 * np.exp(-2.0 * (k / 4.5) ** 2) + 1e-12


def _eps_ref(t):
    return 0.004 + 0.008 * math.exp(-0.5 * (t - 3.0) ** 2)


def _lattice(case, seed, stream):
    lat = Lattice((case["nz"], case["ny"], case["nx"]), case["storage"], case["op"], case["tau"], stream=stream)
    if case.get("domain", "periodic") != "periodic":
        lat.set_domain(case["domain"])
    if case["op"] == "nco":
        lat.set_net_weights(_params(case, seed), case["width"], case["act"], case["mlp"], depth=case["depth"])
    if case["op"] == "mrt":
        lat.set_rates([4.0 / 3.0] * 4)
    return lat


def prepare(case, seed):
    stream = torch.cuda.Stream()
    handle = stream.cuda_stream
    kind = case["kind"]
    state = {"kind": kind, "case": case, "stream": stream}
    if kind == "interval":
        lat = _lattice(case, seed, handle)
        lat.init_equilibrium(*_start(case, seed))
        state["lat"] = lat
    elif kind == "forced":
        lat = _lattice(case, seed, handle)
        rho, u = _flow((case["nz"], case["ny"], case["nx"]), seed, 0.05)
        lat.set_forcing(*_modes(case, seed, DRAW_STEPS), *FORCE, phase_rule=case["phase"])
        lat.init_equilibrium(rho.cpu().numpy(), u.cpu().numpy())
        state["lat"] = lat
    elif kind == "snapshot":
        n, nc = case["n"], case["n"] // case["ratio"]
        fine = Lattice((n,) * 3, case["storage"], "bgk", case["tau"], stream=handle)
        coarse = Lattice((nc,) * 3, "f32", "bgk", 0.5 + (case["tau"] - 0.5) / case["ratio"], stream=handle)
        rho, u = _flow((n,) * 3, seed, 0.05)
        fine.init_equilibrium(rho.cpu().numpy(), u.cpu().numpy())
        state.update(fine=fine, coarse=coarse)
    elif kind == "serve":
        state["lats"] = []
        for i, (n, cls) in enumerate(_solves(case)):
            rho, u = _flow((n,) * 3, seed + 100 * i, U0 / 2)
            lat = Lattice((n,) * 3, cls, "nco", _solve_tau(n), stream=handle)
            lat.set_net_weights(inputs.mlp_params(32, seed), 32, "tanh", "f32_mfma" if cls == "f32" else "bf16")
            if cls == "bf16":
                lat.set_stochastic_rounding(True, i)
            lat.init_equilibrium(rho.cpu().numpy(), u.cpu().numpy())
            lat.set_check(50, 1e-3)
            state["lats"].append(lat)
    elif kind == "dissipation":
        rho, u = _start(case, seed)
        state["unroll"] = DissipationUnroll(
            (case["n"],) * 3, case["tau"], rho, u, U0, case["every"] * case["samples"], case["ckpt"], case["every"],
            _eps_ref, t_min=0.0, act=case["act"], mlp=case["mlp"], width=case["width"], stream=handle,
            domain=case["domain"], depth=case["depth"])
    else:
        ks, draws = _modes(case, seed, case["steps"])
        state["unroll"] = Unroll(
            (case["n"],) * 3, case["tau"], ("pop", _training_start(case, seed).cpu().numpy()), case["steps"],
            case["ckpt"], _target_spectrum(case), case["kmin"], case["kmax"],
            forcing=(ks, draws) + FORCE + (case["phase"],), act=case["act"], mlp=case["mlp"], width=case["width"],
            stream=handle)
    if "unroll" in state:
        state["loss"] = make_autograd(state["unroll"])
        state["params"] = torch.nn.Parameter(torch.tensor(_params(case, seed), dtype=torch.float32))
    return state


def _solves(case):
    return [(int(n), cls) for n in case["grids"].split(",") for cls in ("f32", "bf16")]


def _solve_tau(n):
    return inputs.viscosity(n, U0, 400.0)[1]


class _Span:
    """Device memory of a lattice's current populations for torch.  torch
    holds this object as long as a tensor on the memory lives, and it holds
    the lattice, which owns the memory."""

    def __init__(self, lat):
        ptr, _ = lat.device_populations()
        typestr = {"f32": "<f4", "f64": "<f8", "f16": "<f2", "bf16": "<i2"}[lat.storage]
        self.__cuda_array_interface__ = {"data": (ptr, False), "shape": (27,) + lat.shape, "typestr": typestr,
                                         "version": 2}
        self.lattice = lat


def _populations(lat):
    """The lattice's populations in place, as a tensor of the stored type."""
    t = torch.as_tensor(_Span(lat), device="cuda")
    return t.view(torch.bfloat16) if lat.storage == "bf16" else t


def run(state):
    kind, case = state["kind"], state["case"]
    if kind == "interval":
        lat = state["lat"]
        lat.step(case["steps"])
        if case["domain"] == "tgv_octant":
            # A sampled curve: the mean kinetic energy goes to the host.
            return {"f": _populations(lat), "k": float(lat.global_sums()[4] / lat.n)}
        return {"f": _populations(lat)}
    if kind == "forced":
        state["lat"].step(case["steps"])
        return {"f": _populations(state["lat"])}
    if kind == "snapshot":
        spectrum = state["fine"].energy_spectrum()
        state["coarse"].restrict_from(state["fine"])
        return {"E": spectrum, "f": state["coarse"].populations().astype(np.float32)}
    if kind == "serve":
        lats = state["lats"]
        batch_step(lats, [case["steps"]] * len(lats))
        for lat in lats:
            lat.sync()
        return [_populations(lat) for lat in lats]
    p = state["params"]
    p.grad = None
    loss = state["loss"](p)
    loss.backward()
    return {"loss": loss.detach(), "grad": p.grad}


# ------------------------------------------------------------------- work --

def _net_flops(width, depth):
    return 2 * (48 * (27 * width + (depth - 1) * width * width) + 4 * width)


def work(case):
    """Per step a state is read and written once; network products counted
    for the width asked for.  A reverse step: the network's forward values
    again and twice its products (inputs and weights), the recorded state and
    the adjoint in, the adjoint out."""
    kind = case["kind"]
    if kind in ("interval", "forced"):
        n = case["nx"] * case["ny"] * case["nz"] * case["steps"]
        flops = 450.0 + (_net_flops(case["width"], case["depth"]) if case["op"] == "nco" else 0.0)
        extra = 108.0 if kind == "forced" and case["phase"] else 0.0     # the state's modes come before its step
        return {"bytes": n * (54.0 * SIZE[case["storage"]] + extra), "flops": n * flops}
    if kind == "snapshot":
        n3, nc3 = case["n"] ** 3, (case["n"] // case["ratio"]) ** 3
        return {"bytes": 27.0 * SIZE[case["storage"]] * n3 + 27.0 * 12 * nc3,
                "flops": 7.5 * n3 * math.log2(n3) + 110.0 * n3}
    if kind == "serve":
        b = sum(n ** 3 * 54.0 * SIZE[cls] for n, cls in _solves(case))
        return {"bytes": case["steps"] * b,
                "flops": case["steps"] * sum(n ** 3 for n, _ in _solves(case)) * (450.0 + _net_flops(32, 2))}
    n3 = case["n"] ** 3
    steps = case["every"] * case["samples"] if kind == "dissipation" else case["steps"]
    net = _net_flops(case["width"], case.get("depth", 2))
    return {"bytes": n3 * steps * (216.0 + 324.0), "flops": n3 * steps * (4.0 * net + 1500.0)}


# ------------------------------------------------------------------ exact --

class _Model:
    """D3Q27 stream-collide in float64 torch from the paper's definitions;
    populations (27, nz, ny, nx), velocity index c_x fastest."""

    C = [(x, y, z) for z in (-1, 0, 1) for y in (-1, 0, 1) for x in (-1, 0, 1)]
    ROWS = ("", "x", "y", "z", "xx", "xy", "xz", "yy", "yz", "zz", "xxy", "xxz", "xyy", "xyz", "xzz", "yyz", "yzz",
            "xxyy", "xxyz", "xxzz", "xyyz", "xyzz", "yyzz", "xxyyz", "xxyzz", "xyyzz", "xxyyzz")

    def __init__(self, domain="periodic", params=None, width=0, depth=2, act="tanh"):
        def hermite(n, c):
            return (1.0, math.sqrt(3.0) * c, 3.0 * c * c - 1.0)[n]
        m = [[math.prod(hermite(row.count(a), c[i]) for i, a in enumerate("xyz")) for c in self.C]
             for row in self.ROWS]
        self.M = torch.tensor(m, dtype=torch.float64, device="cuda")
        self.Minv = torch.linalg.inv(self.M)
        self.order = [len(r) for r in self.ROWS]
        self.domain, self.params, self.width, self.depth, self.act = domain, params, width, depth, act
        # m^(g) = M Pi_g M^-1 m for the 48 axis permutations with signs.
        self.G = []
        for perm in itertools.permutations(range(3)):
            for sign in itertools.product((1, -1), repeat=3):
                idx = [self.C.index(tuple(sign[i] * c[perm[i]] for i in range(3))) for c in self.C]
                self.G.append(self.M[:, torch.tensor(idx, device="cuda")] @ self.Minv)
        self._fold = None

    @classmethod
    def weights(cls):
        return torch.tensor([math.prod(2.0 / 3.0 if v == 0 else 1.0 / 6.0 for v in c) for c in cls.C],
                            dtype=torch.float64, device="cuda")

    @classmethod
    def equilibrium(cls, rho, u):
        w = cls.weights()
        uu = u.square().sum(0)
        out = []
        for i, c in enumerate(cls.C):
            cu = c[0] * u[0] + c[1] * u[1] + c[2] * u[2]
            out.append(w[i] * rho * (1.0 + 3.0 * cu + 4.5 * cu * cu - 1.5 * uu))
        return torch.stack(out)

    @classmethod
    def macroscopic(cls, f):
        c = torch.tensor(cls.C, dtype=torch.float64, device="cuda")
        rho = f.sum(0)
        return rho, (c.t() @ f.reshape(27, -1)).reshape((3,) + tuple(f.shape[1:])) / rho

    def _fold_index(self, n):
        """Flat (velocity, node) source of every (velocity, node) of the
        reduced cube: the vortex's mirrors and turns bring it back inside."""
        if self._fold is None:
            z, y, x = np.meshgrid(*[np.arange(n)] * 3, indexing="ij")
            src = np.empty((27, n, n, n), dtype=np.int64)
            for i, c in enumerate(self.C):
                s = [x - c[0], y - c[1], z - c[2]]
                v = [np.full(x.shape, t) for t in c]
                for _ in range(2):
                    for a in range(3):
                        neg = s[a] < 0
                        s[a], v[a] = np.where(neg, -1 - s[a], s[a]), np.where(neg, -v[a], v[a])
                    far = s[2] >= n
                    s = [np.where(far, s[1], s[0]), np.where(far, s[0], s[1]), np.where(far, 2 * n - 1 - s[2], s[2])]
                    v = [np.where(far, v[1], v[0]), np.where(far, v[0], v[1]), np.where(far, -v[2], v[2])]
                    far = s[0] >= n
                    s = [np.where(far, s[1], s[0]), np.where(far, 2 * n - 1 - s[0], s[1]), s[2]]
                    v = [np.where(far, v[1], v[0]), np.where(far, -v[0], v[1]), v[2]]
                    far = s[1] >= n
                    s = [np.where(far, 2 * n - 1 - s[1], s[0]), np.where(far, s[0], s[1]), s[2]]
                    v = [np.where(far, -v[1], v[0]), np.where(far, v[0], v[1]), v[2]]
                src[i] = (9 * (v[2] + 1) + 3 * (v[1] + 1) + v[0] + 1) * n ** 3 + (s[2] * n + s[1]) * n + s[0]
            self._fold = torch.from_numpy(src.ravel()).cuda()
        return self._fold

    def stream(self, f):
        if self.domain == "tgv_octant":
            return f.reshape(-1)[self._fold_index(f.shape[1])].reshape(f.shape)
        return torch.stack([torch.roll(f[i], (c[2], c[1], c[0]), (0, 1, 2)) for i, c in enumerate(self.C)])

    def rates(self, m):
        """omega_3..omega_6 of moments m (27, nodes)."""
        sizes, p, pos, layers = [27] + [self.width] * self.depth + [4], self.params, 0, []
        for a, b in zip(sizes[:-1], sizes[1:]):
            layers.append((p[pos:pos + a * b].reshape(a, b), p[pos + a * b:pos + a * b + b]))
            pos += a * b + b
        g = torch.tanh if self.act == "tanh" else torch.relu
        total = 0.0
        for G in self.G:
            h = (G @ m).t()
            for W, b in layers[:-1]:
                h = g(h @ W + b)
            total = total + h
        W, b = layers[-1]
        t = (total / len(self.G)) @ W + b
        return (1.0 / (0.5 / (1.0 + torch.exp(t)) + 0.5)).t()

    def collide(self, f, op, tau, force=None):
        shape = f.shape
        f = f.reshape(27, -1)
        rho, u = self.macroscopic(f)
        feq = self.equilibrium(rho, u)
        if op == "bgk":
            out = f - (f - feq) / tau
        else:
            m = self.M @ f
            omega = self.rates(m) if op == "nco" else [4.0 / 3.0] * 4
            d = self.M @ (f - feq)
            s = [d[k] * (1.0 if n < 2 else 1.0 / tau if n == 2 else omega[n - 3]) for k, n in enumerate(self.order)]
            out = f - self.Minv @ torch.stack(s)
        if force is not None:
            out = out + self.equilibrium(rho, u + force.reshape(3, -1) / rho) - feq
        return out.reshape(shape)

    def step(self, f, op, tau, force=None):
        f = self.stream(f)
        # Slabs bound the memory of the 48 group elements.
        slab = max(1, (1 << 19) // (f.shape[2] * f.shape[3]))
        parts = [self.collide(f[:, z:z + slab], op, tau, None if force is None else force[:, z:z + slab])
                 for z in range(0, f.shape[1], slab)]
        return torch.cat(parts, 1)

    def force(self, f, ks, draw, phase):
        """Alvelius force of one step on state f: draw (modes, 3) in [0, 1)."""
        amp, kf, c = FORCE
        axes = [2.0 * math.pi * torch.arange(n, dtype=torch.float64, device="cuda") / n for n in f.shape[1:]]
        if phase:
            _, u = self.macroscopic(f)
        total = 0.0
        for k, d in zip(np.asarray(ks, dtype=np.float64), draw):
            kk, kp = math.sqrt((k * k).sum()), math.hypot(k[0], k[1])
            e1 = [k[1] / kp, -k[0] / kp, 0.0] if kp else [1.0, 0.0, 0.0]
            e2 = [k[0] * k[2] / (kk * kp), k[1] * k[2] / (kk * kp), -kp / kk] if kp else [0.0, 1.0, 0.0]
            mag = math.sqrt(amp * math.exp(-(kk - kf) ** 2 / c) / (2.0 * math.pi * kk * kk))
            ga, gb, psi = math.sin(2.0 * math.pi * d[0]), math.cos(2.0 * math.pi * d[0]), 2.0 * math.pi * d[1]
            arg = k[2] * axes[0][:, None, None] + k[1] * axes[1][None, :, None] + k[0] * axes[2][None, None, :]
            cs, sn = torch.cos(arg), torch.sin(arg)
            if phase:
                ur, ui = [(v * cs).mean() for v in u], [-(v * sn).mean() for v in u]
                x1r, x1i = sum(a * b for a, b in zip(ur, e1)), sum(a * b for a, b in zip(ui, e1))
                x2r, x2i = sum(a * b for a, b in zip(ur, e2)), sum(a * b for a, b in zip(ui, e2))
                th = torch.atan2(ga * x1r + gb * (math.cos(psi) * x2r + math.sin(psi) * x2i),
                                 -ga * x1i + gb * (math.sin(psi) * x2r - math.cos(psi) * x2i))
            else:
                th = torch.tensor(2.0 * math.pi * d[2], dtype=torch.float64, device="cuda")
            c1, s1, c2, s2 = torch.cos(th), torch.sin(th), torch.cos(th + psi), torch.sin(th + psi)
            total = total + torch.stack([2.0 * mag * ((ga * c1 * e1[i] + gb * c2 * e2[i]) * cs
                                                      - (ga * s1 * e1[i] + gb * s2 * e2[i]) * sn) for i in range(3)])
        return total

    def spectrum(self, f):
        _, u = self.macroscopic(f)
        n = f.shape[1]
        k = torch.fft.fftfreq(n, 1.0 / n, dtype=torch.float64, device="cuda")
        kk = (k[:, None, None] ** 2 + k[None, :, None] ** 2 + k[None, None, :] ** 2).sqrt()
        shell = torch.floor(kk + 0.5).long().reshape(-1)
        e = 0.0
        for c in range(3):
            e = e + 0.5 * (torch.fft.fftn(u[c]) / n ** 3).abs().square().reshape(-1)
        return torch.zeros(n_bins(n), dtype=torch.float64, device="cuda").index_add(0, shell, e)


def _stored(f, storage):
    """Populations as the storage holds them (16-bit: scaled deviations)."""
    if storage in ("f16", "bf16"):
        w = _Model.weights()
        scale = torch.tensor([4.0 ** (1 + sum(abs(v) for v in c)) for c in _Model.C], dtype=torch.float64, device="cuda")
        f = (f - w[:, None, None, None]) * scale[:, None, None, None]
    return f


def _net_model(case, seed, domain="periodic"):
    params = torch.tensor(_params(case, seed), dtype=torch.float64, device="cuda")
    return _Model(domain, params, case["width"], case.get("depth", 2), case["act"])


def exact(case, seed):
    kind = case["kind"]
    with torch.no_grad():
        if kind == "interval":
            rho, u = (torch.from_numpy(a).cuda() for a in _start(case, seed))
            model = _net_model(case, seed, case["domain"]) if case["op"] == "nco" else _Model(case["domain"])
            f = model.equilibrium(rho, u)
            for _ in range(case["steps"]):
                f = model.step(f, case["op"], case["tau"])
            out = {"f": _stored(f, case["storage"])}
            if case["domain"] == "tgv_octant":
                out["k"] = float(0.5 * model.macroscopic(f)[1].square().sum(0).mean())
            return out
        if kind == "forced":
            model = _Model()
            f = model.equilibrium(*_flow((case["nz"], case["ny"], case["nx"]), seed, 0.05))
            ks, draws = _modes(case, seed, DRAW_STEPS)
            for t in range(case["steps"]):
                f = model.step(f, case["op"], case["tau"], model.force(f, ks, draws[t], case["phase"]))
            return {"f": f}
        if kind == "snapshot":
            model, r = _Model(), case["ratio"]
            f = model.equilibrium(*_flow((case["n"],) * 3, seed, 0.05))
            g = model.stream(f)[:, ::r, ::r, ::r]
            feq = model.equilibrium(*model.macroscopic(g))
            tau_c = 0.5 + (case["tau"] - 0.5) / r
            g = feq + (r * tau_c / case["tau"]) * (g - feq)
            back = [torch.roll(g[i], (-c[2], -c[1], -c[0]), (0, 1, 2)) for i, c in enumerate(model.C)]
            return {"E": model.spectrum(f), "f": torch.stack(back)}
        if kind == "serve":
            out = []
            for i, (n, cls) in enumerate(_solves(case)):
                model = _net_model(dict(width=32, act="tanh"), seed)
                f = model.equilibrium(*_flow((n,) * 3, seed + 100 * i, U0 / 2))
                for _ in range(case["steps"]):
                    f = model.step(f, "nco", _solve_tau(n))
                out.append(_stored(f, cls))
            return out
    return _exact_training(case, seed)


def _exact_training(case, seed):
    from torch.utils.checkpoint import checkpoint
    model = _net_model(case, seed, case.get("domain", "periodic"))
    p = model.params.requires_grad_(True)

    def advance(f, p, force):
        model.params = p
        return model.step(f, "nco", case["tau"], force)

    if case["kind"] == "dissipation":
        rho, u = (torch.from_numpy(a).cuda() for a in _start(case, seed))
        f = model.equilibrium(rho, u)
        ks = [0.5 * model.macroscopic(f)[1].square().sum(0).mean()]
        for t in range(case["every"] * case["samples"]):
            f = checkpoint(advance, f, p, None, use_reentrant=False)
            if (t + 1) % case["every"] == 0:
                ks.append(0.5 * model.macroscopic(f)[1].square().sum(0).mean())
        k = torch.stack(ks) / U0 ** 2
        edge = case["n"] * (4 if case["domain"] == "tgv_octant" else 1)
        dt = case["every"] * U0 / (edge / (2.0 * math.pi))
        eps = -(k[2:] - k[:-2]) / (2.0 * dt)
        ref = torch.tensor([_eps_ref((i + 1) * dt) for i in range(len(eps))], dtype=torch.float64, device="cuda")
        loss = (((eps - ref) / ref.abs().max()) ** 2).mean()
    else:
        f = _training_start(case, seed)
        ks, draws = _modes(case, seed, case["steps"])
        for t in range(case["steps"]):
            force = checkpoint(lambda x, t=t: model.force(x, ks, draws[t], case["phase"]), f, use_reentrant=False)
            f = checkpoint(advance, f, p, force, use_reentrant=False)
        lo, hi = case["kmin"], case["kmax"] + 1
        target = torch.from_numpy(_target_spectrum(case)).cuda()
        loss = ((model.spectrum(f)[lo:hi].log() - target[lo:hi].log()) ** 2).mean()
    loss.backward()
    return {"loss": loss.detach(), "grad": p.grad.detach()}
