"""The work that programs have this library do, as cases to time and to check.

Every case goes through the public entry points of ``paper_2209_00806_amd``:
``listed()`` names one case for each use below, ``draw`` gives more of the
same ranges, ``prepare`` makes what a program holds before the call (the
Hamiltonian handle, the states, the operators), ``run`` is the call, and
``exact`` is what it returns, evaluated with plain torch in 64 bits.

A case with ``shape`` "tuned" sets the launch shape that the autotuner picked
for that kind of operator, as a program does that keeps its tuning results
(``tbpm.autotune_cached``); "default" leaves the handle as it was created.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2209_00806_amd import autograd as ag
from paper_2209_00806_amd import inputs, tbpm

BETA = 38.68  # 1/eV, 300 K
TOL = 1e-12

#: launch shapes the autotuner settles on, by precision: two orders per launch
#: for lattices of a few elements per row, the staged pass for wide rows
TUNED = {
    ("sparse", "fp64"): dict(wg_chunks=2, xcd_remap=5, nontemporal=1, unroll=1, staged=0, vec=2, fused=2),
    ("sparse", "fp32"): dict(wg_chunks=2, xcd_remap=5, nontemporal=1, unroll=1, staged=0, vec=4, fused=2),
    ("wide", "fp64"): dict(wg_chunks=2, xcd_remap=3, nontemporal=0, unroll=1, staged=3, vec=2, fused=0),
    ("wide", "fp32"): dict(wg_chunks=2, xcd_remap=4, nontemporal=0, unroll=1, staged=2, vec=4, fused=0),
}


def listed():
    return [
        # the usage example: clean 64 x 64 graphene, one state, 512 samples, and its DOS (bound by launches)
        dict(name="dos_graphene64", kind="dos", lattice="graphene", nx=64, ny=64, disorder=0.0, states=1, steps=512,
             precision="fp64", shape="default"),
        # the first program of the README: disordered 256 x 256 graphene, four states, 1024 samples, no tuning
        dict(name="dos_graphene256", kind="dos", lattice="graphene", nx=256, ny=256, disorder=1.0, states=4,
             steps=1024, precision="fp64", shape="default"),
        # production DOS: disordered 1024 x 1024 graphene, eight states, in the tuned shape; a stretch of 64 time steps
        dict(name="dos_graphene1024", kind="dos", lattice="graphene", nx=1024, ny=1024, disorder=1.0, states=8,
             steps=65, precision="fp64", shape="tuned"),
        # the same in the FP32 recursion
        dict(name="dos_graphene1024_fp32", kind="dos", lattice="graphene", nx=1024, ny=1024, disorder=1.0, states=8,
             steps=65, precision="fp32", shape="tuned"),
        # complex hoppings (a magnetic field), an odd lattice and a state count that is no power of two, no tuning
        dict(name="dos_magnetic", kind="dos", lattice="hofstadter", nx=231, ny=197, disorder=0.5, states=3, steps=257,
             precision="fp64", shape="default"),
        # twisted bilayer: about twenty elements per row, sixteen states, FP32
        dict(name="dos_bilayer_fp32", kind="dos", lattice="bilayer", nx=192, ny=192, disorder=0.0, states=16, steps=65,
             precision="fp32", shape="tuned"),
        # disorder averaging over samples of uneven size in one launch sequence
        dict(name="batch_fp32", kind="batch", members=12, size_lo=1.0e4, size_hi=1.0e5, states=4, steps=257,
             precision="fp32", shape="tuned"),
        # a training step on the DOS: forward, loss gradient, adjoint, gradients of all bonds and on-site energies
        dict(name="gradient_graphene256", kind="gradient", nx=256, ny=256, states=4, steps=193, every=64,
             shape="tuned"),
        # Kubo-Bastin conductivity: 512 moments and the energy integral
        dict(name="kubo_bastin512", kind="kubo", lattice="graphene", nx=512, ny=512, disorder=1.0, states=1,
             moments=512, energies=1024, shape="tuned"),
        # LDOS of eight orbitals by the recursion method
        dict(name="haydock512", kind="haydock", lattice="graphene", nx=512, ny=512, disorder=1.0, states=8,
             iterations=200, energies=4001, shape="default"),
        # optical conductivity at 300 K, real and imaginary parts
        dict(name="optical256", kind="optical", lattice="graphene", nx=256, ny=256, disorder=1.0, states=1, steps=257,
             precision="fp64", shape="default"),
        # quasi-eigenstates at eight energies
        dict(name="quasi256", kind="quasi", lattice="graphene", nx=256, ny=256, disorder=1.0, states=1, steps=129,
             energies=8, precision="fp64", shape="default"),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["dos", "dos", "dos", "dos", "bilayer", "batch", "gradient", "kubo", "haydock", "optical",
                       "quasi"])
    shape = rng.choice(["default", "tuned"])
    precision = rng.choice(["fp64", "fp64", "fp32"])
    disorder = round(rng.uniform(0.0, 2.0), 3)
    if kind == "dos":
        lattice = rng.choice(["graphene", "graphene", "square", "hofstadter"])
        nx, ny = log_int(24, 720), log_int(24, 720)
        if lattice == "hofstadter":
            nx = 7 * max(4, nx // 7)
        states = rng.choice([1, 1, 2, 3, 4, 5, 8, 13, 16])
        cells = nx * ny * states
        steps = min(log_int(48, 1024), max(17, int(2.0e8 / max(cells, 1))))
        return dict(kind="dos", lattice=lattice, nx=nx, ny=ny, disorder=disorder, states=states, steps=steps,
                    precision=precision, shape=shape)
    if kind == "bilayer":
        nx, ny = log_int(20, 192), log_int(20, 192)
        return dict(kind="dos", lattice="bilayer", nx=nx, ny=ny, disorder=0.0, states=rng.choice([1, 4, 7, 8, 16]),
                    steps=rng.randint(17, 65), precision=rng.choice(["fp64", "fp32"]), shape=shape)
    if kind == "batch":
        return dict(kind="batch", members=rng.randint(2, 12), size_lo=float(log_int(500, 10000)),
                    size_hi=float(log_int(20000, 100000)), states=rng.choice([1, 3, 4, 8]), steps=rng.randint(33, 257),
                    precision=precision, shape=shape)
    if kind == "gradient":
        return dict(kind="gradient", nx=log_int(16, 256), ny=log_int(16, 256), states=rng.choice([1, 2, 3, 4]),
                    steps=rng.randint(40, 193), every=rng.choice([16, 32, 64]), shape=shape)
    lattice = rng.choice(["graphene", "square"])
    if kind == "kubo":
        return dict(kind="kubo", lattice=lattice, nx=log_int(32, 512), ny=log_int(32, 512), disorder=disorder,
                    states=rng.choice([1, 1, 2, 3]), moments=rng.randint(48, 300), energies=rng.randint(200, 1024),
                    shape=shape)
    if kind == "haydock":
        return dict(kind="haydock", lattice=lattice, nx=log_int(128, 512), ny=log_int(128, 512), disorder=disorder,
                    states=rng.choice([1, 3, 8, 16]), iterations=rng.randint(20, 100), energies=rng.randint(500, 4001),
                    shape=shape)
    if kind == "optical":
        return dict(kind="optical", lattice=lattice, nx=log_int(32, 256), ny=log_int(32, 256), disorder=disorder,
                    states=rng.choice([1, 2, 3]), steps=rng.randint(64, 257), precision="fp64", shape=shape)
    return dict(kind="quasi", lattice=lattice, nx=log_int(32, 256), ny=log_int(32, 256), disorder=disorder,
                states=rng.choice([1, 2, 3]), steps=rng.randint(33, 129), energies=rng.randint(1, 8),
                precision=precision, shape=shape)


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------

@functools.lru_cache(maxsize=4)
def _geometry(lattice, nx, ny):
    """The lattice without disorder: the pattern, the hoppings and the bond displacements."""
    if lattice == "graphene":
        return inputs.graphene(nx, ny)
    if lattice == "square":
        return inputs.square(nx, ny)
    if lattice == "hofstadter":
        return inputs.hofstadter(nx, ny, 1, 7, t=-2.7)
    return inputs.twisted_bilayer(nx, ny)


@functools.lru_cache(maxsize=2)
def _bond_geometry(nx, ny):
    return inputs.graphene(nx, ny, keep_bonds=True)


@functools.lru_cache(maxsize=4)
def _current(lattice, nx, ny):
    return inputs.current_values(_geometry(lattice, nx, ny), 0)


def _rng(seed):
    return np.random.default_rng(1000003 + seed)


def _states(seed, n, states):
    """Random-phase states of unit norm, [n, states]."""
    g = torch.Generator(device="cuda")
    g.manual_seed(7 + seed)
    theta = torch.rand((n, states), generator=g, device="cuda", dtype=torch.float64) * (2.0 * math.pi)
    return torch.polar(torch.full_like(theta, 1.0 / math.sqrt(n)), theta)


def _operator(case, seed):
    """(lattice, on-site energies, f): f bounds the spectrum."""
    lat = _geometry(case["lattice"], case["nx"], case["ny"])
    onsite = _rng(seed).uniform(-0.5, 0.5, lat.n_orb) * case["disorder"]
    f = {"graphene": 9.0, "square": 12.0, "hofstadter": 12.0, "bilayer": 12.0}[case["lattice"]]
    return lat, onsite, f


def _members(case, seed):
    """The samples of a batch: sizes and kinds belong to the case, disorder and states to the seed."""
    size = np.random.default_rng(case["members"])
    rng = _rng(seed)
    out = []
    for i in range(case["members"]):
        n = math.exp(size.uniform(math.log(case["size_lo"]), math.log(case["size_hi"])))
        if size.uniform() < 0.5:
            side = max(3, int(round(math.sqrt(n / 2.0))))
            lat = inputs.graphene(side, side)
        else:
            side = max(3, int(round(math.sqrt(n))))
            lat = inputs.square(side, side)
        onsite = rng.uniform(-0.5, 0.5, lat.n_orb) * size.uniform(0.0, 2.0)
        out.append((lat, onsite, 9.0 if lat.meta["kind"] == "graphene" else 12.0, _states(seed * 64 + i, lat.n_orb,
                                                                                          case["states"])))
    return out


def _orbitals(case, seed, n):
    return np.sort(_rng(seed + 17).choice(n, size=case["states"], replace=False))


def _energies(case):
    return [-2.5 + 0.71 * j for j in range(case["energies"])]


def _shape(h, case, rows="sparse"):
    if case["shape"] == "tuned":
        for precision in ("fp64", "fp32"):
            h.set_launch_config(precision=precision, **TUNED[(rows, precision)])


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        members = _members(case, seed)
        hams = [tbpm.Hamiltonian(lat.n_orb, lat.row_ptr, lat.col, lat.val, onsite) for lat, onsite, _, _ in members]
        batch = tbpm.Batch(hams)
        _shape(batch, case)
        fs = [f for _, _, f, _ in members]
        return dict(case=case, batch=batch, states=[psi for _, _, _, psi in members], dt=[math.pi / f for f in fs],
                    f=fs)
    if kind == "gradient":
        lat = _bond_geometry(case["nx"], case["ny"])
        h = tbpm.Hamiltonian(lat.n_orb, lat.row_ptr, lat.col, lat.val, lat.onsite)
        _shape(h, case)
        return dict(case=case, h=h, nnz=lat.nnz, slots=(torch.from_numpy(lat.slot_ij).cuda(),
                                                        torch.from_numpy(lat.slot_ji).cuda()),
                    **_gradient_inputs(case, seed, lat))
    lat, onsite, f = _operator(case, seed)
    h = tbpm.Hamiltonian(lat.n_orb, lat.row_ptr, lat.col, lat.val, onsite)
    _shape(h, case, "wide" if case["lattice"] == "bilayer" else "sparse")
    state = dict(case=case, h=h, f=f, dt=math.pi / f)
    if kind == "haydock":
        psi = torch.zeros((lat.n_orb, case["states"]), dtype=torch.complex128, device="cuda")
        at = torch.from_numpy(_orbitals(case, seed, lat.n_orb)).cuda()
        psi[at, torch.arange(case["states"], device="cuda")] = 1.0
        state["psi"] = psi
        state["energies"] = torch.linspace(-10.0, 10.0, case["energies"], dtype=torch.float64, device="cuda")
    else:
        state["psi"] = _states(seed, lat.n_orb, case["states"])
    if kind in ("kubo", "optical"):
        state["current"] = _current(case["lattice"], case["nx"], case["ny"])
        state["area"] = lat.area / lat.n_orb
    if kind == "kubo":
        state["mus"] = torch.linspace(-3.0, 3.0, 25, dtype=torch.float64, device="cuda")
    return state


def _gradient_inputs(case, seed, lat):
    rng = _rng(seed)
    t = torch.from_numpy(-2.7 * (1.0 + 0.05 * rng.standard_normal(lat.bond_i.shape[0]))).cuda()
    target = torch.from_numpy(rng.uniform(0.0, 0.2, 2 * case["steps"])).cuda()
    return dict(t=t, eps=torch.zeros(lat.n_orb, dtype=torch.float64, device="cuda"),
                psi=_states(seed, lat.n_orb, case["states"]), target=target, f=9.0, dt=math.pi / 9.0)


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "dos":
        corr = tbpm.propagate(s["h"], s["psi"], case["steps"], s["dt"], s["f"], precision=case["precision"])
        energies, dos = tbpm.dos(corr, s["dt"])
        return dict(corr=corr, energies=energies, dos=dos)
    if kind == "batch":
        return s["batch"].propagate(s["states"], case["steps"], s["dt"], s["f"], precision=case["precision"])
    if kind == "gradient":
        t = s["t"].detach().requires_grad_(True)
        eps = s["eps"].detach().requires_grad_(True)
        val = ag.bond_values(s["nnz"], s["slots"][0], s["slots"][1], t)
        _, dos = ag.tbpm_dos(s["h"], val, eps, s["psi"], case["steps"], s["dt"], s["f"], ckpt_every=case["every"])
        loss = torch.sum((dos[::8] - s["target"][::8]) ** 2)
        loss.backward()
        return dict(dos=dos.detach(), t=t.grad, eps=eps.grad)
    if kind == "kubo":
        mu = tbpm.kpm_moments(s["h"], s["current"], s["current"], s["psi"], case["moments"], s["f"])
        sigma, energies, weight = tbpm.kubo_bastin(mu, s["f"], -0.98 * s["f"], 0.98 * s["f"], case["energies"], BETA,
                                                   s["mus"], s["area"])
        return dict(mu=mu, sigma=sigma, energies=energies, weight=weight)
    if kind == "haydock":
        a, b = tbpm.haydock(s["h"], s["psi"], case["iterations"])
        return dict(a=a, b=b, ldos=tbpm.haydock_ldos(a, b, s["energies"], 0.02))
    if kind == "optical":
        corr = tbpm.ac_corr(s["h"], s["current"], s["current"], s["psi"], case["steps"], s["dt"], BETA, 0.0,
                            rescale=s["f"], precision=case["precision"])
        omega, re = tbpm.ac_cond(corr, s["dt"], BETA, s["area"])
        return dict(corr=corr, omega=omega, re=re, im=tbpm.ac_cond_imag(re))
    return dict(states=tbpm.quasi_eigenstates(s["h"], s["psi"], _energies(case), case["steps"], s["dt"], s["f"],
                                              precision=case["precision"]))


# --------------------------------------------------------------------------
# what a pass cannot do without
# --------------------------------------------------------------------------

def _sizes(case):
    """(orbitals, stored elements, flops of one multiply-add with an element)."""
    if case["kind"] == "gradient":
        n = 2 * case["nx"] * case["ny"]
        return n, 3 * n, 4
    cells = case["nx"] * case["ny"]
    if case["lattice"] == "graphene":
        return 2 * cells, 6 * cells, 4
    if case["lattice"] == "bilayer":
        return 4 * cells, 77 * cells, 4
    return cells, 4 * cells, 8 if case["lattice"] == "hofstadter" else 4


def work(case):
    """The inputs read once and the outputs written once; the multiply-adds of the series."""
    kind = case["kind"]
    orders = 17  # sparse products per time step at f dt = pi
    if kind == "batch":
        n = case["members"] * (case["size_hi"] - case["size_lo"]) / math.log(case["size_hi"] / case["size_lo"])
        S, steps = case["states"], case["steps"]
        return dict(bytes=n * (16.0 * S + 3.5 * 12.0 + 8.0) + 16.0 * S * steps * case["members"],
                    flops=orders * (steps - 1) * n * S * (4.0 * 4.5 + 12.0))
    n, nnz, per = _sizes(case)
    S = case["states"]
    matrix = nnz * (4.0 + 2.0 * per) + 8.0 * n
    product = S * (per * nnz + 16.0 * n)  # one product and the recurrence's update
    if kind == "dos":
        steps = case["steps"]
        return dict(bytes=matrix + 16.0 * n * S + 16.0 * S * steps + 32.0 * steps,
                    flops=orders * (steps - 1) * product + 8.0 * steps * steps)
    if kind == "gradient":
        return dict(bytes=matrix + 16.0 * n * S + 12.0 * nnz + 16.0 * n, flops=3.0 * orders * (case["steps"] - 1) * product)
    if kind == "kubo":
        M = case["moments"]
        return dict(bytes=matrix + 16.0 * nnz + 16.0 * n * S + 16.0 * M * M,
                    flops=3.0 * M * product + 8.0 * M * M * n * S + 12.0 * case["energies"] * M * M)
    if kind == "haydock":
        k = case["iterations"]
        return dict(bytes=matrix + 16.0 * n * S + 16.0 * k * S + 8.0 * S * case["energies"], flops=k * (product + 16.0 * n * S))
    if kind == "optical":
        series = 2600
        return dict(bytes=matrix + 16.0 * nnz + 16.0 * n * S + 16.0 * S * case["steps"],
                    flops=2.0 * (series + orders * case["steps"]) * product)
    E = case["energies"]
    return dict(bytes=matrix + 16.0 * n * S + 16.0 * n * S * E,
                flops=2.0 * (case["steps"] - 1) * (orders * product + 8.0 * n * S * E))


# --------------------------------------------------------------------------
# the same in 64 bits with plain torch
# --------------------------------------------------------------------------

class _Matrix:
    """H as padded rows of (column, value)."""

    def __init__(self, lat, val, onsite):
        n = lat.n_orb
        counts = np.diff(lat.row_ptr)
        width = int(counts.max())
        rows = np.repeat(np.arange(n), counts)
        k = np.arange(lat.nnz) - lat.row_ptr[rows]
        col = np.tile(np.arange(n, dtype=np.int64)[:, None], (1, width))
        col[rows, k] = lat.col
        v = np.zeros((n, width), dtype=np.complex128)
        v[rows, k] = val
        v = v if np.any(v.imag) else v.real.copy()
        self.at = [torch.from_numpy(np.ascontiguousarray(col[:, q])).cuda() for q in range(width)]
        self.v = [torch.from_numpy(np.ascontiguousarray(v[:, q])).cuda()[:, None] for q in range(width)]
        self.e = torch.from_numpy(np.asarray(onsite)).cuda()[:, None]

    def __call__(self, x):
        y = self.e * x
        for at, v in zip(self.at, self.v):
            y += v * x[at]
        return y


def _bessel(z, m):
    """J_0(z) .. J_{m-1}(z) by the trapezoidal rule on Bessel's integral (periodic: exact to rounding)."""
    th = np.arange(256) * (2.0 * math.pi / 256)
    return [float(np.mean(np.cos(k * th - z * np.sin(th)))) for k in range(m)]


def _step(H, f, dt, sign=1.0):
    """psi -> exp(-i sign H dt) psi by the Chebyshev series."""
    J = _bessel(f * dt, 24)

    def advance(psi):
        t0, t1 = psi, H(psi) / f
        out = J[0] * t0 + (-2j * sign * J[1]) * t1
        for m in range(2, 24):
            t0, t1 = t1, (2.0 / f) * H(t1) - t0
            out += (2.0 * J[m] * (-1j * sign) ** m) * t1
        return out

    return advance


def _hann(n):
    k = torch.arange(n, dtype=torch.float64, device="cuda")
    return 0.5 * (1.0 + torch.cos(math.pi * k / n))


def _phases(n, count):
    """e^{i pi j k / n} for j = -n .. n-1 (rows) and k < count, the angle reduced in whole numbers."""
    j = torch.arange(-n, n, device="cuda")[:, None]
    k = torch.arange(count, device="cuda")[None, :]
    a = ((j * k) % (2 * n)).to(torch.float64) * (math.pi / n)
    return torch.polar(torch.ones_like(a), a)


def _dos(corr, dt):
    n = corr.shape[0]
    w = _hann(n) * 2.0
    w[0] = 1.0
    c = corr.mean(dim=1) * w
    energies = torch.arange(-n, n, dtype=torch.float64, device="cuda") * (math.pi / (n * dt))
    return energies, (_phases(n, n) @ c[:, None])[:, 0].real * (dt / (2.0 * math.pi))


def _correlation(H, f, dt, psi0, steps):
    advance, psi, corr = _step(H, f, dt), psi0, []
    for k in range(steps):
        if k:
            psi = advance(psi)
        corr.append((psi0.conj() * psi).sum(dim=0))
    return torch.stack(corr)


class _Product(torch.autograd.Function):
    """y = H x for real symmetric values v [n, width], differentiable in v, the on-site energies and x."""

    @staticmethod
    def forward(ctx, x, v, e, at):
        ctx.save_for_backward(x, v, e, at)
        y = e[:, None] * x
        for q in range(at.shape[1]):
            y += v[:, q, None] * x[at[:, q]]
        return y

    @staticmethod
    def backward(ctx, g):
        x, v, e, at = ctx.saved_tensors
        gx = e[:, None] * g
        gv = torch.empty_like(v)
        for q in range(at.shape[1]):
            gx += v[:, q, None] * g[at[:, q]]
            gv[:, q] = (g * x[at[:, q]].conj()).real.sum(dim=1)
        return gx, gv, (g * x.conj()).real.sum(dim=1), None


def _exact_gradient(case, seed):
    lat = _bond_geometry(case["nx"], case["ny"])
    s = _gradient_inputs(case, seed, lat)
    n, f, dt, steps, psi0 = lat.n_orb, s["f"], s["dt"], case["steps"], s["psi"]
    if np.any(np.diff(lat.row_ptr) != 3):
        return None
    at = torch.from_numpy(lat.col.reshape(n, 3).astype(np.int64)).cuda()
    slot = torch.empty(3 * n, dtype=torch.int64, device="cuda")
    bonds = torch.arange(lat.bond_i.shape[0], device="cuda")
    slot[torch.from_numpy(lat.slot_ij).cuda()] = bonds
    slot[torch.from_numpy(lat.slot_ji).cuda()] = bonds
    v, e = s["t"][slot].reshape(n, 3), s["eps"]
    J = _bessel(f * dt, 24)

    def advance(psi, v, e):
        t0, t1 = psi, _Product.apply(psi, v, e, at) / f
        out = J[0] * t0 + (-2j * J[1]) * t1
        for m in range(2, 24):
            t0, t1 = t1, (2.0 / f) * _Product.apply(t1, v, e, at) - t0
            out = out + (2.0 * J[m] * (-1j) ** m) * t1
        return out

    psis = [psi0]
    with torch.no_grad():
        for _ in range(steps - 1):
            psis.append(advance(psis[-1], v, e))
        corr = torch.stack([(psi0.conj() * p).sum(dim=0) for p in psis])
    c = corr.requires_grad_(True)
    _, dos = _dos(c, dt)
    gc, = torch.autograd.grad(torch.sum((dos[::8] - s["target"][::8]) ** 2), c)
    gv, ge, lam = torch.zeros_like(v), torch.zeros_like(e), torch.zeros_like(psi0)
    for k in range(steps - 1, 0, -1):
        lam = lam + gc[k] * psi0
        x, vv, ee = (t.detach().requires_grad_(True) for t in (psis[k - 1], v, e))
        lam, dv, de = torch.autograd.grad(advance(x, vv, ee), (x, vv, ee), lam)
        gv += dv
        ge += de
    gt = torch.zeros_like(s["t"]).index_add_(0, slot, gv.reshape(-1))
    return dict(dos=dos.detach(), t=gt, eps=ge)


def _exact_kubo(case, lat, H, f, psi):
    M, S = case["moments"], case["states"]
    V = _Matrix(lat, _current(case["lattice"], case["nx"], case["ny"]), np.zeros(lat.n_orb))

    def chebyshev(x):
        t0, t1 = x, H(x) / f
        for m in range(M):
            yield t0
            t0, t1 = t1, (2.0 / f) * H(t1) - t0

    L = torch.stack([t.reshape(-1) for t in chebyshev(V(psi))])
    mu = torch.empty((M, M), dtype=torch.complex128, device="cuda")
    for n, t in enumerate(chebyshev(psi)):
        mu[:, n] = (L.conj() @ V(t).reshape(-1, 1))[:, 0] / S
    del L
    m = torch.arange(M, dtype=torch.float64, device="cuda")
    q = math.pi / (M + 1)
    g = ((M - m + 1) * torch.cos(q * m) + torch.sin(q * m) / math.tan(q)) / (M + 1)
    g[0] *= 0.5
    lo, hi = math.acos(0.98), math.acos(-0.98)
    d = (hi - lo) / case["energies"]
    th = lo + (torch.arange(case["energies"], dtype=torch.float64, device="cuda") + 0.5) * d
    x, sn = torch.cos(th), torch.sin(th)
    mt = mu * g[:, None] * g[None, :]
    c = torch.cos(m[:, None] * th[None, :])
    ph = torch.polar(torch.ones_like(c), m[:, None] * th[None, :])
    p = (x[None, :] - 1j * m[:, None] * sn[None, :]) * ph
    F = (c * (mt @ p) + p.conj() * (mt @ c.to(torch.complex128))).sum(dim=0).real
    weight = F * sn * d / ((1.0 - x) * (1.0 + x)) ** 2
    mus = torch.linspace(-3.0, 3.0, 25, dtype=torch.float64, device="cuda")
    fd = 0.5 * (1.0 - torch.tanh(0.5 * BETA * (f * x[None, :] - mus[:, None])))
    sigma = 4.0 / (math.pi * (lat.area / lat.n_orb) * f * f) * (fd * weight[None, :]).sum(dim=1)
    return dict(mu=mu, sigma=sigma, energies=f * x, weight=weight)


def _exact_haydock(case, seed, lat, H):
    n, S = lat.n_orb, case["states"]
    u = torch.zeros((n, S), dtype=torch.complex128, device="cuda")
    u[torch.from_numpy(_orbitals(case, seed, n)).cuda(), torch.arange(S, device="cuda")] = 1.0
    prev, b, As, Bs = torch.zeros_like(u), torch.zeros(S, dtype=torch.float64, device="cuda"), [], []
    for _ in range(case["iterations"]):
        y = H(u) - b * prev
        a = (u.conj() * y).sum(dim=0).real
        y -= a * u
        b = torch.sqrt((y.real ** 2 + y.imag ** 2).sum(dim=0))
        prev, u = u, y / b
        As.append(a)
        Bs.append(b)
    a, b = torch.stack(As), torch.stack(Bs)
    z = torch.linspace(-10.0, 10.0, case["energies"], dtype=torch.float64, device="cuda")[:, None] + 0.02j
    t = z - a[-1]
    for q in range(case["iterations"] - 2, -1, -1):
        t = z - a[q] - b[q] ** 2 / t
    return dict(a=a, b=b, ldos=-(1.0 / t).imag / math.pi)


def _exact_optical(case, lat, H, f, dt, psi):
    S, steps = case["states"], case["steps"]
    V = _Matrix(lat, _current(case["lattice"], case["nx"], case["ny"]), np.zeros(lat.n_orb))
    N = 65536
    x = f * torch.cos(2.0 * math.pi * torch.arange(N, dtype=torch.float64, device="cuda") / N)
    a = torch.fft.fft(0.5 * (1.0 - torch.tanh(0.5 * BETA * x))).real[: N // 2] * (2.0 / N)
    a[0] *= 0.5
    a = a[: int(torch.nonzero(a.abs() >= 1e-14).max()) + 1].tolist()
    blk = torch.cat([V(psi), psi], dim=1)
    t0, t1 = blk, H(blk) / f
    out = a[0] * t0 + a[1] * t1
    for ak in a[2:]:
        t0, t1 = t1, (2.0 / f) * H(t1) - t0
        out += ak * t1
    psi12 = torch.cat([blk[:, :S] - out[:, :S], out[:, S:]], dim=1)
    advance, corr = _step(H, f, dt), []
    for k in range(steps):
        if k:
            psi12 = advance(psi12)
        corr.append((psi12[:, S:].conj() * V(psi12[:, :S].contiguous())).sum(dim=0))
    corr = torch.stack(corr)
    j = torch.arange(steps, dtype=torch.float64, device="cuda")
    omega = math.pi * j / (steps * dt)
    c = corr.mean(dim=1).imag * _hann(steps) * 2.0
    c[0] = 0.0
    s = (_phases(steps, steps)[steps:].imag @ c[:, None])[:, 0]
    w = torch.where(j > 0, omega, torch.ones_like(omega))
    re = torch.where(j > 0, (torch.exp(-BETA * w) - 1.0) / (w * (lat.area / lat.n_orb)) * s * dt, torch.zeros_like(s))
    # principal value of the piecewise linear, even extension of Re sigma: one closed-form weight per grid point

    def xlogx(u):
        return torch.where(u == 0, torch.zeros_like(u), u * torch.log(u.abs().clamp_min(1e-300)))

    m = torch.arange(-2 * steps, 2 * steps + 1, dtype=torch.float64, device="cuda")
    g = xlogx(1.0 - m) - xlogx(1.0 + m) + 2.0 * xlogx(m)
    big = m.abs() >= 2
    mb = torch.where(big, m.abs(), torch.full_like(m, 2.0))
    g = torch.where(big, torch.sign(m) * (-mb * torch.log1p(-1.0 / (mb * mb)) - torch.log1p(2.0 / (mb - 1.0))), g)
    k, q = torch.arange(steps, device="cuda")[:, None], torch.arange(steps, device="cuda")[None, :]
    K = g[k - q + 2 * steps] + torch.where(q > 0, g[k + q + 2 * steps], torch.zeros((), dtype=g.dtype, device="cuda"))
    return dict(corr=corr, omega=omega, re=re, im=-(K @ re) / math.pi)


def _exact_quasi(case, H, f, dt, psi0):
    energies, w = _energies(case), _hann(case["steps"]).tolist()
    acc = torch.zeros((len(energies),) + tuple(psi0.shape), dtype=torch.complex128, device="cuda")
    for sign in (1.0, -1.0):
        advance, psi = _step(H, f, dt, sign), psi0
        for k in range(case["steps"]):
            if k:
                psi = advance(psi)
            elif sign < 0:
                continue
            for j, e in enumerate(energies):
                acc[j] += (w[k] * complex(math.cos(e * k * dt), sign * math.sin(e * k * dt))) * psi
    return dict(states=acc / torch.sqrt((acc.real ** 2 + acc.imag ** 2).sum(dim=1, keepdim=True)))


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        return [_correlation(_Matrix(lat, lat.val, onsite), f, math.pi / f, psi, case["steps"])
                for lat, onsite, f, psi in _members(case, seed)]
    if kind == "gradient":
        return _exact_gradient(case, seed)
    lat, onsite, f = _operator(case, seed)
    dt, H = math.pi / f, _Matrix(lat, lat.val, onsite)
    if kind == "haydock":
        return _exact_haydock(case, seed, lat, H)
    psi = _states(seed, lat.n_orb, case["states"])
    if kind == "dos":
        corr = _correlation(H, f, dt, psi, case["steps"])
        energies, dos = _dos(corr, dt)
        return dict(corr=corr, energies=energies, dos=dos)
    if kind == "kubo":
        return _exact_kubo(case, lat, H, f, psi)
    if kind == "optical":
        return _exact_optical(case, lat, H, f, dt, psi)
    return _exact_quasi(case, H, f, dt, psi)
