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
