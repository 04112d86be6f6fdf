"""Several Clenshaw orders per launch (rows of at most four stored elements)
against one order per launch and the oracle, where tiles, shells, blocks of
states and launch sequences end.

Bars: against the one-order kernels, FP64 correlations to 1e-12 of their largest
value (a few thousand operations of rounding 1e-16, in another order), and
FP32-mixed ones to 1e-12 as well: the FP32 states are the same bit for bit, and
only their FP64 sums run in another order.  Against the oracle 1e-10 (FP64)."""
import math

import numpy as np
import pytest

import oracle
from paper_2209_00806_amd import inputs, tbpm

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CHAIN = dict(wg_chunks=2, xcd_remap=5, nontemporal=1, unroll=1, staged=0, vec=2, fused=2)


def _rel(a, b):
    return float(np.max(np.abs(a - b)) / np.max(np.abs(b)))


def _cplx(lat, rng):
    i = np.repeat(np.arange(lat.n_orb), np.diff(lat.row_ptr))
    a = rng.uniform(0, 2 * np.pi, lat.n_orb)
    lat.val = lat.val * np.exp(1j * (a[i] - a[lat.col]))
    return lat


def _lattice(kind, rng):
    lat = {
        "ring5": lambda: inputs.from_bonds(5, np.arange(5), (np.arange(5) + 1) % 5, np.full(5, -2.7), np.zeros(5)),
        "graphene_small": lambda: inputs.graphene(23, 19),  # tiles follow an order of their own
        "graphene": lambda: inputs.graphene(113, 89),  # renumbered, several tiles, ragged sizes
        "square_open": lambda: inputs.square(61, 47, pbc=False),  # rows of 2 to 4 elements
        "graphene_complex": lambda: _cplx(inputs.graphene(41, 37), rng),
        "square_complex": lambda: _cplx(inputs.square(45, 53), rng),
    }[kind]()
    lat.onsite = inputs.anderson(rng, lat.n_orb, 1.0)
    return lat


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("kind", ["ring5", "graphene_small", "graphene", "square_open", "graphene_complex",
                                  "square_complex"])
def test_chain_matches_one_order_per_launch(kind, precision):
    rng = np.random.default_rng(3)
    lat = _lattice(kind, rng)
    f = 1.05 * oracle.gershgorin(lat.row_ptr, lat.val, lat.onsite)
    H = tbpm.Hamiltonian.from_lattice(lat)
    # states: one, odd counts (padded blocks), more than one workgroup's share;
    # dt f = pi (17 orders), 0.3 (few orders, one launch), 9 (many launches);
    # 35 samples: whole graphs and a remainder
    for S, z, nt in ((1, math.pi, 35), (3, math.pi, 18), (8, 0.3, 9), (5, 9.0, 5), (1, 1e-7, 4)):
        psi_np = inputs.random_phase_states(rng, lat.n_orb, S)
        psi = torch.from_numpy(psi_np).cuda()
        H.set_launch_config()
        ref, n_ref = tbpm.propagate(H, psi, nt, z / f, f, precision=precision, return_norm=True)
        H.set_launch_config(**CHAIN)
        for graph in (True, False):
            got, n_got = tbpm.propagate(H, psi, nt, z / f, f, precision=precision, return_norm=True, graph=graph)
            assert _rel(got.cpu().numpy(), ref.cpu().numpy()) < 1e-12, (S, z, nt, graph)
            assert _rel(n_got.cpu().numpy(), n_ref.cpu().numpy()) < 1e-12, (S, z, nt, graph)
        if precision == "fp64":
            want, _, _ = oracle.propagate(lat.row_ptr, lat.col, lat.val, lat.onsite, psi_np, nt, z / f, f)
            assert _rel(got.cpu().numpy(), want) < 1e-10, (S, z, nt)
    H.close()


@pytest.mark.parametrize("kind", ["graphene_small", "graphene", "square_complex"])
def test_chain_stored_states(kind):
    """Checkpoints, snapshots and quasi-eigenstates (states leave the blocks in the caller's order)."""
    rng = np.random.default_rng(4)
    lat = _lattice(kind, rng)
    f = 1.05 * oracle.gershgorin(lat.row_ptr, lat.val, lat.onsite)
    dt = math.pi / f
    H = tbpm.Hamiltonian.from_lattice(lat)
    for S in (1, 3):
        psi = torch.from_numpy(inputs.random_phase_states(rng, lat.n_orb, S)).cuda()
        out = []
        for shape in ({}, CHAIN):
            H.set_launch_config(**shape)
            _, ck = tbpm.propagate(H, psi, 23, dt, f, ckpt_every=5)
            out.append([ck, tbpm.propagate_snapshots(H, psi, [19, 0, 2], dt, f),
                        tbpm.propagate_snapshots(H, psi, [18, 3], dt, f, precision="fp32"),
                        tbpm.quasi_eigenstates(H, psi, [-0.7, 1.1], 20, dt, f)])
        for a, b in zip(*out):
            assert _rel(b.cpu().numpy(), a.cpu().numpy()) < 1e-12
    H.close()


def test_chain_without_a_configuration():
    """A handle nobody configured takes several orders per launch for long runs, with current values and in
    batches of members below and above a tile; configured handles keep their shape."""
    rng = np.random.default_rng(5)
    lats = [_lattice(k, rng) for k in ("ring5", "graphene_small", "graphene", "square_open")]
    fs = [1.05 * oracle.gershgorin(l.row_ptr, l.val, l.onsite) for l in lats]
    psis = [torch.from_numpy(inputs.random_phase_states(rng, l.n_orb, 2)).cuda() for l in lats]
    hams = [tbpm.Hamiltonian.from_lattice(l) for l in lats]
    for precision in ("fp64", "fp32"):
        B = tbpm.Batch(hams)
        got = B.propagate(psis, 70, [math.pi / f for f in fs], fs, precision=precision)
        B.set_launch_config()
        ref = B.propagate(psis, 70, [math.pi / f for f in fs], fs, precision=precision)
        for a, b in zip(got, ref):
            assert _rel(a.cpu().numpy(), b.cpu().numpy()) < 1e-11
        B.close()
    lat, H, psi, f = lats[2], hams[2], psis[2], fs[2]
    first = tbpm.propagate(H, psi, 70, math.pi / f, f)
    on = torch.from_numpy(lat.onsite * 0.5).cuda()
    H.set_values(torch.from_numpy(lat.val * 0.9).cuda(), on)
    got = tbpm.propagate(H, psi, 70, math.pi / f, f)
    H.set_launch_config()
    ref = tbpm.propagate(H, psi, 70, math.pi / f, f)
    assert _rel(got.cpu().numpy(), ref.cpu().numpy()) < 1e-11
    assert _rel(first.cpu().numpy(), ref.cpu().numpy()) > 1e-3  # the values did change


@pytest.mark.parametrize("kind", ["ring5", "graphene_small", "graphene", "square_open", "graphene_complex",
                                  "square_complex", "chain5"])
def test_chain_backward_matches_one_order_per_launch(kind):
    """The replay that stores every order and the adjoint's several orders per launch (chain5, six elements per
    row: the two-order launches).  A gradient is a sum of some 1e5 products of states with errors of 1e-14 against
    each other: 1e-11 of the largest gradient, and 1e-10 against the oracle."""
    rng = np.random.default_rng(6)
    if kind == "chain5":
        i = np.arange(300)
        lat = inputs.from_bonds(300, np.concatenate([i, i, i]), np.concatenate([(i + d) % 300 for d in (1, 2, 7)]),
                                -1.0 - rng.random(900), rng.uniform(-1, 1, 300))
    else:
        lat = _lattice(kind, rng)
    f = 1.05 * oracle.gershgorin(lat.row_ptr, lat.val, lat.onsite)
    H = tbpm.Hamiltonian.from_lattice(lat)
    # one, odd and many states (groups of blocks); 17, few and many orders; segments with a remainder
    for S, z, nt, K in ((1, math.pi, 12, 4), (3, math.pi, 8, 3), (8, 0.3, 6, 8), (5, 9.0, 4, 2), (2, 1e-7, 3, 1)):
        psi_np = inputs.random_phase_states(rng, lat.n_orb, S)
        psi = torch.from_numpy(psi_np).cuda()
        g = rng.standard_normal((nt, S)) + 1j * rng.standard_normal((nt, S))
        gd = torch.from_numpy(g).cuda()
        out = []
        for shape in ({}, CHAIN):
            H.set_launch_config(**shape)
            _, ck = tbpm.propagate(H, psi, nt, z / f, f, ckpt_every=K)
            out.append([t.cpu().numpy() for t in tbpm.backward(H, psi, nt, z / f, f, gd, K, ck)])
        for a, b in zip(*out):
            assert _rel(b, a) < 1e-11, (S, z, nt)
        if lat.n_orb < 10000:
            for b, w in zip(out[1], oracle.backward(lat.row_ptr, lat.col, lat.val, lat.onsite, psi_np, nt, z / f, f, g)):
                assert _rel(b if H.info()["is_complex"] else b.real, w if H.info()["is_complex"] else w.real) < 1e-10
    H.close()


@pytest.mark.parametrize("kind", ["graphene_small", "graphene", "square_open", "graphene_complex", "square_complex"])
def test_chain_moments_match_one_order_per_launch(kind):
    """Kubo-Bastin moments with several Chebyshev orders per launch and the current operator applied in them:
    fewest moments, one block of moments and a remainder, odd state counts.  A moment sums products of vectors
    with errors of M 1e-16: 1e-12 of the largest moment."""
    rng = np.random.default_rng(7)
    lat = _lattice(kind, rng)
    f = 1.05 * oracle.gershgorin(lat.row_ptr, lat.val, lat.onsite)
    if kind.startswith("graphene"):
        ja, jb = inputs.current_values(lat, 0), inputs.current_values(lat, 1)
    else:  # any antisymmetric displacements
        i = np.repeat(np.arange(lat.n_orb), np.diff(lat.row_ptr))
        x = rng.uniform(0, 1, lat.n_orb)
        ja = 1j * lat.val * (x[lat.col] - x[i])
        jb = 1j * lat.val * (np.sin(9 * x)[lat.col] - np.sin(9 * x)[i])
    H = tbpm.Hamiltonian.from_lattice(lat)
    for S, M in ((1, 2), (1, 3), (3, 4), (2, 130), (1, 261)):
        psi = torch.from_numpy(inputs.random_phase_states(rng, lat.n_orb, S)).cuda()
        out = []
        for shape in ({}, CHAIN):
            H.set_launch_config(**shape)
            out.append(tbpm.kpm_moments(H, ja, jb, psi, M, f).cpu().numpy())
        assert _rel(out[1], out[0]) < 1e-12, (S, M)
    H.close()


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n_steps", [2, 8, 9, 17, 18, 27, 41])
def test_chain_accumulates_several_steps_per_launch(n_steps, precision):
    """Quasi-eigenstates and current correlations take the states of up to eight steps per launch: runs that end
    within a group of steps, at its end, within a graph and after it, against one step at a time (one order per
    launch).  Sums of n_steps terms of rounding 1e-16: 1e-12."""
    rng = np.random.default_rng(8)
    lat = _lattice("graphene_small", rng)
    f = 1.05 * oracle.gershgorin(lat.row_ptr, lat.val, lat.onsite)
    dt = math.pi / f
    J = inputs.current_values(lat, 0)
    H = tbpm.Hamiltonian.from_lattice(lat)
    psi = torch.from_numpy(inputs.random_phase_states(rng, lat.n_orb, 3)).cuda()
    out = []
    for shape in ({}, CHAIN):
        H.set_launch_config(**shape, precision=precision)
        out.append([tbpm.quasi_eigenstates(H, psi, [-0.7, 1.1, 2.3], n_steps, dt, f, precision=precision),
                    tbpm.ac_corr(H, J, J, psi, n_steps, dt, 10.0, 0.1, rescale=f, precision=precision)])
    for a, b in zip(*out):
        assert _rel(b.cpu().numpy(), a.cpu().numpy()) < 1e-12
    H.close()


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("nx,ny,band", [(9, 7, 0), (23, 21, 0), (67, 61, 0), (0, 5000, 3), (0, 5000, 5), (0, 5000, 7),
                                        (0, 5000, 9)])
def test_chain_wide_rows(nx, ny, band, precision):
    """The wide pass of real operators with rows of 5 to 24 elements (bilayers, and bands of 6, 10, 14 and 18
    elements for the other table widths) against the general one: bars as above."""
    rng = np.random.default_rng(9)
    if nx:
        lat = inputs.twisted_bilayer(nx, ny)
    else:
        i = np.arange(ny)
        lat = inputs.from_bonds(ny, np.concatenate([i] * band), np.concatenate([(i + d + 1) % ny for d in range(band)]),
                                -0.2 - rng.random(ny * band), np.zeros(ny))
    lat.onsite = inputs.anderson(rng, lat.n_orb, 1.0)
    f = 1.05 * oracle.gershgorin(lat.row_ptr, lat.val, lat.onsite)
    H = tbpm.Hamiltonian.from_lattice(lat)
    for S, z, nt in ((1, math.pi, 19), (3, math.pi, 6), (16, math.pi, 4), (8, 0.3, 9), (5, 9.0, 3), (2, 1e-7, 3)):
        psi = torch.from_numpy(inputs.random_phase_states(rng, lat.n_orb, S)).cuda()
        H.set_launch_config()
        ref, n_ref = tbpm.propagate(H, psi, nt, z / f, f, precision=precision, return_norm=True)
        for shape in (CHAIN, dict(wg_chunks=2, xcd_remap=3, nontemporal=0, unroll=1, staged=2, vec=4, fused=0)):
            H.set_launch_config(**shape)
            got, n_got = tbpm.propagate(H, psi, nt, z / f, f, precision=precision, return_norm=True)
            assert _rel(got.cpu().numpy(), ref.cpu().numpy()) < 1e-12, (S, z, nt)
            assert _rel(n_got.cpu().numpy(), n_ref.cpu().numpy()) < 1e-12, (S, z, nt)
    H.close()


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("nx,far", [(9, 0), (17, 1), (31, 0)])
def test_wide_rows_in_any_order(nx, far, precision):
    """The wide pass takes its tiles from the caller's order where that is local and from an order of its own where
    it is not: bilayers with their rows shuffled, all of them or (far) every 16th, against the general pass."""
    rng = np.random.default_rng(12)
    lat = inputs.twisted_bilayer(nx, nx)
    n = lat.n_orb
    perm = np.arange(n)
    moved = np.arange(0, n, 16) if far else np.arange(n)
    perm[moved] = rng.permutation(moved)
    i = np.repeat(np.arange(n), np.diff(lat.row_ptr))
    up = i < lat.col
    lat = inputs.from_bonds(n, perm[i[up]], perm[lat.col[up]], lat.val[up], inputs.anderson(rng, n, 1.0))
    f = 1.05 * oracle.gershgorin(lat.row_ptr, lat.val, lat.onsite)
    H = tbpm.Hamiltonian.from_lattice(lat)
    for S, nt in ((8, 9), (3, 4)):
        psi = torch.from_numpy(inputs.random_phase_states(rng, n, S)).cuda()
        out = []
        for shape in ({}, dict(wg_chunks=2, xcd_remap=3, nontemporal=0, unroll=1, staged=2, vec=4, fused=0)):
            H.set_launch_config(**shape)
            out.append(tbpm.propagate(H, psi, nt, math.pi / f, f, precision=precision))
        assert _rel(out[1].cpu().numpy(), out[0].cpu().numpy()) < 1e-12
    H.close()


@pytest.mark.parametrize("kind", ["ring5", "graphene_small", "graphene", "square_open", "graphene_complex",
                                  "square_complex"])
def test_chain_haydock_one_launch_per_iteration(kind):
    """Lanczos coefficients with one launch per iteration against the two-launch form: odd state counts, start
    vectors that span an invariant subspace (the ring: exact zeros after its fifth iteration) and a zero one,
    lengths within and beyond a graph.  Both forms round differently, which the recursion amplifies slowly: 1e-9
    of the Gershgorin bound over 50 iterations; graph and direct launches bit for bit."""
    rng = np.random.default_rng(10)
    lat = _lattice(kind, rng)
    H = tbpm.Hamiltonian.from_lattice(lat)
    g = H.info()["gershgorin"]
    for S, n_iter in ((1, 50), (3, 13), (8, 29), (5, 1), (2, 6)):
        st = inputs.random_phase_states(rng, lat.n_orb, S)
        st[:, S - 1] = 0.0
        st[:, 0] = 0.0
        st[lat.n_orb // 2, 0] = 1.0
        psi = torch.from_numpy(st).cuda()
        H.set_launch_config()
        a, b = (t.cpu().numpy() for t in tbpm.haydock(H, psi, n_iter))
        H.set_launch_config(**CHAIN)
        a1, b1 = (t.cpu().numpy() for t in tbpm.haydock(H, psi, n_iter))
        a2, b2 = (t.cpu().numpy() for t in tbpm.haydock(H, psi, n_iter, graph=False))
        assert np.array_equal(a1, a2) and np.array_equal(b1, b2)
        m = min(n_iter, 4) if kind == "ring5" else n_iter  # what follows an exhausted subspace is rounding
        assert np.max(np.abs(a1[:m] - a[:m])) < 1e-9 * g and np.max(np.abs(b1[:m] - b[:m])) < 1e-9 * g
        if S > 1:
            assert not a1[:, S - 1].any() and not b1[:, S - 1].any()
        if kind == "ring5" and n_iter > 6:
            assert not b1[5:, 0].any() and not a1[6:, 0].any()
    H.close()


def test_wide_rows_stored_states_and_batch():
    """The wide pass with checkpoints, snapshots, quasi-eigenstates and current correlations (states leave the
    blocks in the caller's order), and in a batch of members of uneven size: 1e-12 against one order per launch."""
    rng = np.random.default_rng(11)
    staged = dict(wg_chunks=2, xcd_remap=3, nontemporal=0, unroll=1, staged=2, vec=4, fused=0)
    lats = [inputs.twisted_bilayer(n, n) for n in (7, 23, 12)]
    for lat in lats:
        lat.onsite = inputs.anderson(rng, lat.n_orb, 1.0)
    fs = [1.05 * oracle.gershgorin(lat.row_ptr, lat.val, lat.onsite) for lat in lats]
    hams = [tbpm.Hamiltonian.from_lattice(lat) for lat in lats]
    H, lat, f = hams[1], lats[1], fs[1]
    dt = math.pi / f
    i = np.repeat(np.arange(lat.n_orb), np.diff(lat.row_ptr))
    x = rng.uniform(0, 1, lat.n_orb)
    J = 1j * lat.val * (x[lat.col] - x[i])
    for S in (3, 6):
        psi = torch.from_numpy(inputs.random_phase_states(rng, lat.n_orb, S)).cuda()
        out = []
        for shape in ({}, staged):
            H.set_launch_config(**shape)
            _, ck = tbpm.propagate(H, psi, 23, dt, f, ckpt_every=5)
            out.append([ck, tbpm.propagate_snapshots(H, psi, [19, 0, 2], dt, f),
                        tbpm.propagate_snapshots(H, psi, [18, 3], dt, f, precision="fp32"),
                        tbpm.quasi_eigenstates(H, psi, [-0.7, 1.1], 20, dt, f),
                        tbpm.quasi_eigenstates(H, psi, [0.4], 9, dt, f, precision="fp32"),
                        tbpm.ac_corr(H, J, J, psi, 19, dt, 10.0, 0.1, rescale=f)])
        for a, b in zip(*out):
            assert _rel(b.cpu().numpy(), a.cpu().numpy()) < 1e-12
    B = tbpm.Batch(hams)
    psis = [torch.from_numpy(inputs.random_phase_states(rng, l.n_orb, 5)).cuda() for l in lats]
    for precision in ("fp64", "fp32"):
        out = []
        for shape in ({}, staged):
            B.set_launch_config(**shape)
            out.append(B.propagate(psis, 21, [math.pi / v for v in fs], fs, precision=precision))
        for a, b in zip(*out):
            assert _rel(b.cpu().numpy(), a.cpu().numpy()) < 1e-12
