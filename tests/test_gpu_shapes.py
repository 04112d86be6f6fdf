"""Launch shapes that only some operators, sizes or sequences of calls reach."""
import math

import numpy as np
import pytest

import oracle
from paper_2209_00806_amd import inputs, tbpm

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("M,n_e", [(3, 5), (256, 4097), (590, 4096), (591, 4096), (1097, 5), (1098, 7), (2048, 3),
                                   (2049, 3), (4096, 2)])
def test_kubo_bastin_energies_per_workgroup(M, n_e):
    """One, two and four energies per workgroup, where the rule and the LDS of each end, against the sum over both
    indices in factored form.  The phases m theta are good to M 1e-16, the sums of M^2 random terms to less of
    their size: 1e-10 of the largest conductivity."""
    rng = np.random.default_rng(M + n_e)
    mu = rng.standard_normal((M, M)) + 1j * rng.standard_normal((M, M))
    mus = np.linspace(-6.0, 6.0, 9)
    f, lo, hi, beta, area = 9.0, -8.0, 7.9, 4.0, 3.0
    sg, en, _ = tbpm.kubo_bastin(_dev(mu), f, lo, hi, n_e, beta, mus, area)
    w = oracle.jackson(M) / np.where(np.arange(M) == 0, 2.0, 1.0)
    t0, t1 = np.arccos(hi / f), np.arccos(lo / f)
    th = t0 + (np.arange(n_e) + 0.5) * (t1 - t0) / n_e
    x, s, m = np.cos(th)[:, None], np.sin(th)[:, None], np.arange(M)[None, :]
    c = w * np.cos(m * th[:, None])
    p = w * (x - 1j * m * s) * np.exp(1j * m * th[:, None])
    q = w * (x + 1j * m * s) * np.exp(-1j * m * th[:, None])
    val = (np.sum(c * (p @ mu.T), axis=1) + np.sum(q * (c @ mu.T), axis=1)).real / (1.0 - x[:, 0] ** 2) ** 2
    fd = oracle.fermi(f * x, beta, mus[None, :])
    ref = 4.0 / (np.pi * area * f * f) * np.sum(fd * (val * s[:, 0] * (t1 - t0) / n_e)[:, None], axis=0)
    assert np.max(np.abs(sg.cpu().numpy() - ref)) < 1e-10 * np.max(np.abs(ref))
    np.testing.assert_allclose(en.cpu().numpy(), f * x[:, 0], rtol=0, atol=1e-13)


def _rel(a, b):
    return float(np.max(np.abs(a - b)) / np.max(np.abs(b)))


def _band(n, hops, rng, periodic=True):
    """n rows, each joined to the rows at the given distances (2 len(hops) elements per row)."""
    i = np.arange(n)
    bi = np.concatenate([i] * len(hops))
    bj = np.concatenate([i + h for h in hops])
    keep = np.ones(bj.size, bool) if periodic else bj < n
    return inputs.from_bonds(n, bi[keep], bj[keep] % n, -0.2 - rng.random(int(keep.sum())), inputs.anderson(rng, n, 1.0))


STAGED = dict(wg_chunks=2, xcd_remap=3, nontemporal=0, unroll=1, staged=2, vec=2, fused=0)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("hops,periodic", [(3, True), (3, False), (4, True), (5, False), (6, True), (7, True), (8, False),
                                           (9, True), (10, True), (11, True), (12, True), (12, False)])
def test_wide_pass_at_every_table_width(hops, periodic, precision):
    """The wide pass with tables of 6 to 24 elements per row (full rows, and open ends with shorter ones) against
    the general pass: 1e-12 of the largest correlation, some thousand operations of rounding 1e-16 in another
    order; FP32 states are the same bit for bit."""
    rng = np.random.default_rng(hops)
    lat = _band(1500, range(1, hops + 1), rng, periodic)
    f = 1.05 * oracle.gershgorin(lat.row_ptr, lat.val, lat.onsite)
    H = tbpm.Hamiltonian.from_lattice(lat)
    for S, nt in ((4, 18), (7, 3)):
        psi = _dev(inputs.random_phase_states(rng, lat.n_orb, S))
        out = []
        for shape in ({}, STAGED):
            H.set_launch_config(**shape, precision=precision)
            out.append(tbpm.propagate(H, psi, nt, math.pi / f, f, precision=precision).cpu().numpy())
        assert _rel(out[1], out[0]) < 1e-12, (S, nt)
    H.close()


def _six(n, rng, cplx=False):
    """Six elements per row, in three distances: the launches of two orders take them (fused), as they take any
    operator of more than four elements that is not the wide pass's."""
    lat = _band(n, (1, 2, 7), rng)
    if cplx:
        i = np.repeat(np.arange(n), np.diff(lat.row_ptr))
        a = rng.uniform(0, 2 * np.pi, n)
        lat.val = lat.val * np.exp(1j * (a[i] - a[lat.col]))
    return lat


def _dt_for_terms(f, terms):
    return next(z for z in np.geomspace(1e-3, 12.0, 4000) if tbpm.num_terms(z) == terms) / f


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("cplx", [False, True])
@pytest.mark.parametrize("terms", [5, 6, 7, 17, 18])
def test_pairs_of_orders(terms, cplx, precision):
    """The schedule of two orders per launch, on rows that the chain does not take: the shortest series that pair
    the last orders, both parities of the middle ones, graphs and their remainders, stored states (the last order
    alone), 1, 2 and 4 states per thread.  FP64: 1e-13 of the largest correlation against one order per launch,
    the same arithmetic in other tiles, and 1e-10 against the oracle; FP32 states carry errors of some 1e-6."""
    rng = np.random.default_rng(terms)
    lat = _six(700, rng, cplx)
    S = 5
    psi = inputs.random_phase_states(rng, lat.n_orb, S)
    f = 1.05 * oracle.gershgorin(lat.row_ptr, lat.val, lat.onsite)
    dt = _dt_for_terms(f, terms)
    H = tbpm.Hamiltonian.from_lattice(lat)
    for tier, vec, nt in ((1, 1, 2), (2, 2, 17), (4, 4, 35), (6, 2, 35)):
        H.set_launch_config(2, 1, 1, 1, vec=vec, precision=precision, fused=0)
        plain = tbpm.propagate(H, _dev(psi), nt, dt, f, precision=precision).cpu().numpy()
        H.set_launch_config(2, 1, 1, 1, vec=vec, precision=precision, fused=tier)
        got = tbpm.propagate(H, _dev(psi), nt, dt, f, precision=precision).cpu().numpy()
        nog = tbpm.propagate(H, _dev(psi), nt, dt, f, precision=precision, graph=False).cpu().numpy()
        bar = 1e-13 if precision == "fp64" else 1e-5
        assert _rel(got, plain) < bar and _rel(nog, plain) < bar, (tier, nt)
        if precision == "fp64":
            ck, _ = tbpm.propagate(H, _dev(psi), nt, dt, f, ckpt_every=4)
            assert _rel(ck.cpu().numpy(), plain) < bar, (tier, nt)
    ref, _, _ = oracle.propagate(lat.row_ptr, lat.col, lat.val, lat.onsite, psi, nt, dt, f)
    assert _rel(got, ref) < (1e-10 if precision == "fp64" else 1e-5)
    H.close()


@pytest.mark.parametrize("terms", [9, 11, 18])
@pytest.mark.parametrize("tier,vec", [(1, 1), (2, 2), (4, 4), (3, 2)])
@pytest.mark.parametrize("cplx", [False, True])
def test_pairs_of_adjoint_orders(cplx, tier, vec, terms):
    """The gradient with replay and adjoint two orders per launch (first pair, middle pairs, single orders left, the
    last order; 1, 2 or 4 states per thread), on rows that the chain does not take, against the oracle's adjoint
    (1e-10) and one order per launch (1e-12)."""
    rng = np.random.default_rng(23)
    lat = _six(150, rng, cplx)
    S, nt = 5, 19
    psi = inputs.random_phase_states(rng, lat.n_orb, S)
    f = 1.05 * oracle.gershgorin(lat.row_ptr, lat.val, lat.onsite)
    dt = _dt_for_terms(f, terms)
    g = rng.standard_normal((nt, S)) + 1j * rng.standard_normal((nt, S))
    gv, go = oracle.backward(lat.row_ptr, lat.col, lat.val, lat.onsite, psi, nt, dt, f, g)
    H = tbpm.Hamiltonian.from_lattice(lat)
    out = []
    for fused in (0, tier):
        H.set_launch_config(2, 1, 1, 1, vec=vec if fused else 1, precision="fp64", fused=fused)
        _, ck = tbpm.propagate(H, _dev(psi), nt, dt, f, ckpt_every=5)
        out.append([t.cpu().numpy() for t in tbpm.backward(H, _dev(psi), nt, dt, f, _dev(g), 5, ck)])
    a = out[1][0] if cplx else out[1][0].real
    assert _rel(a, gv if cplx else gv.real) < 1e-10 and _rel(out[1][1], go) < 1e-10
    assert _rel(out[1][0], out[0][0]) < 1e-12 and _rel(out[1][1], out[0][1]) < 1e-12
    H.close()


@pytest.mark.parametrize("cplx", [False, True])
@pytest.mark.parametrize("S,M", [(1, 4), (3, 5), (2, 64), (5, 131)])
def test_pairs_of_moment_orders(S, M, cplx):
    """Both Chebyshev recursions of the Kubo moments two orders per launch, on rows that the chain does not take:
    fewest moments, odd counts, more than one block of them, against the oracle (1e-11 of the largest moment) and
    one order per launch (1e-12)."""
    rng = np.random.default_rng(M)
    lat = _six(400, rng, cplx)
    i = np.repeat(np.arange(lat.n_orb), np.diff(lat.row_ptr))
    x = rng.uniform(0, 1, lat.n_orb)
    ja, jb = 1j * lat.val * (x[lat.col] - x[i]), 1j * lat.val * (np.sin(9 * x)[lat.col] - np.sin(9 * x)[i])
    psi = inputs.random_phase_states(rng, lat.n_orb, S)
    f = 1.05 * oracle.gershgorin(lat.row_ptr, lat.val, lat.onsite)
    ref = oracle.kpm_moments(lat.row_ptr, lat.col, lat.val, lat.onsite, ja, jb, psi, M, f)
    H = tbpm.Hamiltonian.from_lattice(lat)
    out = []
    for fused in (0, 2):
        H.set_launch_config(2, 1, 1, 1, vec=2 if fused else 1, precision="fp64", fused=fused)
        out.append(tbpm.kpm_moments(H, ja, jb, _dev(psi), M, f).cpu().numpy())
    assert _rel(out[1], ref) < 1e-11 and _rel(out[1], out[0]) < 1e-12
    H.close()


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("cplx", [False, True])
@pytest.mark.parametrize("beta", [0.05, 3.0, 20.0])
def test_pairs_of_fermi_orders(beta, cplx, precision):
    """The Fermi series two orders per launch, on rows that the chain does not take: few and many terms, through
    the optical correlation against the oracle (1e-10; FP32 propagation 2e-5) and one order per launch (1e-12)."""
    rng = np.random.default_rng(31)
    lat = _six(300, rng, cplx)
    i = np.repeat(np.arange(lat.n_orb), np.diff(lat.row_ptr))
    x = rng.uniform(0, 1, lat.n_orb)
    J = 1j * lat.val * (x[lat.col] - x[i])
    psi = inputs.random_phase_states(rng, lat.n_orb, 3)
    f = 1.05 * oracle.gershgorin(lat.row_ptr, lat.val, lat.onsite)
    dt = math.pi / f
    ref, _, _ = oracle.ac_corr(lat.row_ptr, lat.col, lat.val, lat.onsite, J, J, psi, 20, dt, f, beta, 0.1,
                               fermi_tol=1e-13)
    H = tbpm.Hamiltonian.from_lattice(lat)
    out = []
    for fused in (0, 2):
        H.set_launch_config(2, 1, 1, 1, vec=2, precision="fp64", fused=fused)
        out.append(tbpm.ac_corr(H, J, J, _dev(psi), 20, dt, beta, 0.1, rescale=f, fermi_tol=1e-13,
                                precision=precision).cpu().numpy())
    assert _rel(out[1], ref) < (1e-10 if precision == "fp64" else 2e-5)
    assert _rel(out[1], out[0]) < (1e-12 if precision == "fp64" else 2e-5)
    H.close()


@pytest.mark.parametrize("kind", ["graphene", "square_complex", "bilayer"])
@pytest.mark.parametrize("configured", [False, True])
def test_calls_of_all_kinds_in_turn_on_one_handle(kind, configured):
    """Calls that differ in method, state count, time step, length and precision, in two orders on one handle, give
    what each gives on a handle of its own: 1e-13 of its largest value."""
    rng = np.random.default_rng(41)
    lat = {"graphene": lambda: inputs.graphene(41, 37), "square_complex": lambda: inputs.square(45, 43),
           "bilayer": lambda: inputs.twisted_bilayer(17, 17)}[kind]()
    lat.onsite = inputs.anderson(rng, lat.n_orb, 1.0)
    if kind == "square_complex":
        i = np.repeat(np.arange(lat.n_orb), np.diff(lat.row_ptr))
        a = rng.uniform(0, 2 * np.pi, lat.n_orb)
        lat.val = lat.val * np.exp(1j * (a[i] - a[lat.col]))
    i = np.repeat(np.arange(lat.n_orb), np.diff(lat.row_ptr))
    x = rng.uniform(0, 1, lat.n_orb)
    J = 1j * lat.val * (x[lat.col] - x[i])
    f = 1.05 * oracle.gershgorin(lat.row_ptr, lat.val, lat.onsite)
    psi = {S: _dev(inputs.random_phase_states(rng, lat.n_orb, S)) for S in (1, 2, 3, 8)}
    g = _dev(rng.standard_normal((66, 2)) + 1j * rng.standard_normal((66, 2)))
    ck = tbpm.Hamiltonian.from_lattice(lat)
    _, ckpt = tbpm.propagate(ck, psi[2], 66, 1.0 / f, f, ckpt_every=16)
    ck.close()
    calls = {
        "long": lambda H: tbpm.propagate(H, psi[1], 70, math.pi / f, f),
        "wide": lambda H: tbpm.propagate(H, psi[8], 70, math.pi / f, f),
        "short steps": lambda H: tbpm.propagate(H, psi[3], 70, 0.3 / f, f),
        "fp32": lambda H: tbpm.propagate(H, psi[8], 66, math.pi / f, f, precision="fp32"),
        "few": lambda H: tbpm.propagate(H, psi[8], 5, 6.0 / f, f),
        "haydock": lambda H: tbpm.haydock(H, psi[3], 70)[0],
        "moments": lambda H: tbpm.kpm_moments(H, J, J, psi[2], 150, f),
        "optical": lambda H: tbpm.ac_corr(H, J, J, psi[2], 66, 0.5 / f, 5.0, 0.1, rescale=f),
        "quasi": lambda H: tbpm.quasi_eigenstates(H, psi[3], [-0.7, 1.1], 66, math.pi / f, f),
        "gradient": lambda H: tbpm.backward(H, psi[2], 66, 1.0 / f, f, g, 16, ckpt)[0],
    }

    def handle():
        H = tbpm.Hamiltonian.from_lattice(lat)
        if configured:
            for p in ("fp64", "fp32"):
                if kind == "bilayer":
                    H.set_launch_config(**STAGED, precision=p)
                else:
                    H.set_launch_config(2, 5, 1, 1, vec=2, precision=p, fused=2)
        return H

    want = {}
    for name, call in calls.items():
        H = handle()
        want[name] = call(H).cpu().numpy()
        H.close()
    H = handle()
    names = list(calls)
    for name in names + [names[k] for k in rng.permutation(len(names))] + names[::-1]:
        assert _rel(calls[name](H).cpu().numpy(), want[name]) < 1e-13, name
    H.close()
