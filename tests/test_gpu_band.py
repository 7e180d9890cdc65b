"""Parity of the GPU Band_DFT_Col Part 5 (chemical potential, band energy,
occupations) and Part 6 (charge and energy density matrices) with the
oracle, through the C ABI.

Tolerances.  mu: both sides bisect the same count function in FP64 but sum
it in different orders, so a decision can differ where the count is within
rounding of nelec; the resulting mu difference is bounded by that rounding
(a few ulp of the count, taken as 1e-13 * nelec) divided by the slope
dN/dmu = g sum wk f (1 - f) / kT, plus the final bracket width.  The band
energy and the occupations move by the slopes times that bound.  Density
matrices: each entry is a sum of K = nk * nocc products; the bound is
8 K u times the sum of the magnitudes of its terms."""
import numpy as np
import pytest
import torch

import oracle as O
from gpu_helpers import DEV, K, check, dev, host
from paper_1402_4247_amd import inputs as G

pytestmark = pytest.mark.gpu
U = np.finfo(np.float64).eps / 2


def gpu_fermi(w, wk, nelec, kT, g):
    kg = K()
    nk, n = w.shape
    dw = torch.from_numpy(np.ascontiguousarray(w)).to(DEV)
    dwk = torch.from_numpy(np.ascontiguousarray(wk, dtype=np.float64)).to(DEV)
    occ = torch.full((nk, n), -1.0, dtype=torch.float64, device=DEV)
    res = torch.zeros(3, dtype=torch.float64, device=DEV)
    st = torch.full((1,), -7, dtype=torch.int32, device=DEV)
    with kg.Context(0) as ctx:
        check(kg.fermi_device(ctx, dw, n, nk, dwk, nelec, kT, g, occ, res, st), "fermi_device")
        torch.cuda.synchronize()
    return res.cpu().numpy(), occ.cpu().numpy(), int(st.cpu().numpy()[0])


def mu_tolerance(w, wk, occ, nelec, kT, g, mu):
    slope = g * float((np.asarray(wk)[:, None] * occ * (1.0 - occ)).sum()) / kT
    return 1e-13 * nelec / max(slope, 1e-300) + 8 * U * max(1.0, abs(mu)), slope


@pytest.mark.parametrize("nk,n,kT,fill", [(1, 1, 0.05, 0.3), (4, 300, 0.02, 0.5), (3, 1100, 0.2, 0.37),
                                         (16, 777, 0.005, 0.61)])
def test_fermi_matches_oracle(nk, n, kT, fill):
    rng = np.random.default_rng(1000 + n)
    w = np.sort(rng.standard_normal((nk, n)), axis=1)
    wk = rng.uniform(0.5, 1.5, nk)
    wk /= wk.sum()
    g = 2.0
    nelec = fill * g * n
    mu0, eb0, cnt0, occ0 = O.fermi(w, wk, nelec, kT, g)
    res, occ, st = gpu_fermi(w, wk, nelec, kT, g)
    assert st == 0
    tol, slope = mu_tolerance(w, wk, occ0, nelec, kT, g, mu0)
    dmu = abs(res[0] - mu0)
    assert dmu <= tol, (dmu, tol)
    sumabs = g * float((wk[:, None] * np.abs(w)).sum())
    assert abs(res[1] - eb0) <= (sumabs / kT) * dmu + 64 * U * sumabs * n
    assert abs(res[2] - nelec) <= slope * dmu + 1e-12 * nelec
    assert np.abs(occ - occ0).max() <= dmu / (4 * kT) + 64 * U


# where Newton steps start badly: nearly empty and nearly full bands, levels far
# apart on the scale of kT, one that is wide against the spectrum
@pytest.mark.parametrize("nk,n,kT,fill", [(1, 1, 1e-3, 0.01), (2, 64, 0.05, 1e-6), (2, 1025, 3.0, 0.999),
                                          (4, 300, 1e-4, 0.5), (5, 90, 0.01, 0.995)])
def test_fermi_newton_edges(nk, n, kT, fill):
    test_fermi_matches_oracle(nk, n, kT, fill)


def test_fermi_in_a_gap():
    # the count is flat there: mu is anywhere inside, the occupations are 0 or 1
    # to the rounding of the count (n terms of one)
    rng = np.random.default_rng(77)
    nk, n = 3, 130
    w = np.sort(np.where(np.arange(n) < n // 2, -1.0, 1.0) + rng.uniform(-0.1, 0.1, (nk, n)), axis=1)
    res, occ, st = gpu_fermi(w, np.full(nk, 1.0 / nk), float(n), 0.01, 2.0)
    assert st == 0 and -0.9 < res[0] < 0.9
    assert abs(res[2] - n) <= 1e-12 * n
    assert np.abs(occ - (w < 0)).max() <= 1e-12 * n


def test_fermi_out_of_range_status():
    w = np.array([[-1.0, 0.0, 1.0]])
    for nelec in (0.0, 6.0, 7.5, -1.0):
        res, occ, st = gpu_fermi(w, [1.0], nelec, 0.1, 2.0)
        assert st == 4          # KGEV_ERANGE
        assert np.all(occ == -1.0)


def test_fermi_argument_errors():
    kg = K()
    d = torch.zeros((1, 4), dtype=torch.float64, device=DEV)
    wk = torch.ones(1, dtype=torch.float64, device=DEV)
    res = torch.zeros(3, dtype=torch.float64, device=DEV)
    st = torch.zeros(1, dtype=torch.int32, device=DEV)
    with kg.Context(0) as ctx:
        assert kg.fermi_device(ctx, d, 4, 1, wk, 2.0, 0.0, 2.0, None, res, st) == -8
        assert kg.fermi_device(ctx, d, 4, 1, wk, 2.0, 0.1, 0.0, None, res, st) == -9
        assert kg.fermi_device(ctx, d, 0, 1, wk, 2.0, 0.1, 2.0, None, res, st) == -4
        assert kg.fermi_device(ctx, d, 4, 1, wk, 2.0, 0.1, 2.0, None, None, st) == -12
        assert kg.fermi_device(ctx, d, 4, 1, wk, 2.0, 0.1, 2.0, None, res, None) == -13


def gpu_density(Ccol, w, occ, wk, g, nocc, edm=True, ldr=None):
    kg = K()
    nk, n, _ = Ccol.shape
    dC = torch.from_numpy(np.ascontiguousarray(Ccol)).to(DEV)
    dw = torch.from_numpy(np.ascontiguousarray(w)).to(DEV)
    docc = torch.from_numpy(np.ascontiguousarray(occ)).to(DEV)
    dwk = torch.from_numpy(np.ascontiguousarray(wk, dtype=np.float64)).to(DEV)
    ldr = n if ldr is None else ldr
    sentinel = complex(7.0, -3.0)
    rho = torch.full((n, ldr), sentinel, dtype=torch.complex128, device=DEV)
    E = torch.full((n, ldr), sentinel, dtype=torch.complex128, device=DEV) if edm else None
    with kg.Context(0) as ctx:
        check(kg.density_device(ctx, dC, n, nk, nocc, dw, docc, dwk, g, rho, E, ldr=ldr), "density_device")
        torch.cuda.synchronize()
    # buffers are column-major with ld ldr: row index fastest
    r = rho.cpu().numpy()[:, :n].T
    e = E.cpu().numpy()[:, :n].T if edm else None
    return r, e, sentinel


def density_bound(C, occ, w, wk, g, nocc):
    A = np.abs(C[:, :, :nocc])
    f = (np.asarray(wk)[:, None] * occ[:, :nocc])
    rb = g * np.einsum("kaj,kbj,kj->ab", A, A, f)
    eb = g * np.einsum("kaj,kbj,kj->ab", A, A, f * np.abs(w[:, :nocc]))
    K_ = C.shape[0] * nocc
    return 8 * K_ * U * rb + 1e-300, 8 * K_ * U * eb + 1e-300


@pytest.mark.parametrize("nk,n,nocc,ldr", [(1, 1, 1, 1), (3, 150, 100, 150), (2, 257, 257, 300), (4, 64, 0, 64),
                                           (5, 130, 77, 131)])
def test_density_matches_oracle(nk, n, nocc, ldr):
    rng = np.random.default_rng(2000 + n)
    C = (rng.standard_normal((nk, n, n)) + 1j * rng.standard_normal((nk, n, n))) / np.sqrt(n)
    w = np.sort(rng.standard_normal((nk, n)), axis=1)
    occ = rng.uniform(0, 1, (nk, n))
    wk = rng.uniform(0.5, 1.5, nk)
    wk /= wk.sum()
    g = 2.0
    rho0, E0 = O.density(C, w, occ, wk, g, nocc=nocc)
    r, e, sentinel = gpu_density(np.swapaxes(C, 1, 2), w, occ, wk, g, nocc, ldr=ldr)
    rb, eb = density_bound(C, occ, w, wk, g, nocc)
    low = np.tril(np.ones((n, n), dtype=bool))
    assert np.all(np.abs(r - rho0)[low] <= rb[low])
    assert np.all(np.abs(e - E0)[low] <= eb[low])
    # the strict upper triangle is left untouched
    up = ~low
    assert np.all(r[up] == sentinel) and np.all(e[up] == sentinel)


def test_density_without_edm():
    rng = np.random.default_rng(9)
    nk, n = 2, 90
    C = (rng.standard_normal((nk, n, n)) + 1j * rng.standard_normal((nk, n, n))) / np.sqrt(n)
    w = np.sort(rng.standard_normal((nk, n)), axis=1)
    occ = rng.uniform(0, 1, (nk, n))
    rho0, _ = O.density(C, w, occ, [0.5, 0.5], 1.0, edm=False)
    r, e, _ = gpu_density(np.swapaxes(C, 1, 2), w, occ, [0.5, 0.5], 1.0, n, edm=False)
    rb, _ = density_bound(C, occ, w, [0.5, 0.5], 1.0, n)
    low = np.tril(np.ones((n, n), dtype=bool))
    assert np.all(np.abs(r - rho0)[low] <= rb[low])


def test_solve_fermi_density_chain():
    # Parts 2-6 on the device: the S-trace of rho counts the electrons and
    # the S-trace of edm is the band energy (C_k^H S C_k = I)
    kg = K()
    n, nk = 200, 3
    kpts = G.mp_grid(4)[:nk]
    Hs, Ss = G.lcao_batch(n, kpts, 77)
    dH, dS = dev(Hs), dev(Ss)
    dw = torch.zeros((nk, n), dtype=torch.float64, device=DEV)
    dC = torch.zeros((nk, n, n), dtype=torch.complex128, device=DEV)
    wk = torch.full((nk,), 1.0 / nk, dtype=torch.float64, device=DEV)
    occ = torch.zeros((nk, n), dtype=torch.float64, device=DEV)
    res = torch.zeros(3, dtype=torch.float64, device=DEV)
    st = torch.zeros(1, dtype=torch.int32, device=DEV)
    rho = torch.zeros((n, n), dtype=torch.complex128, device=DEV)
    E = torch.zeros((n, n), dtype=torch.complex128, device=DEV)
    nelec = 0.8 * n
    with kg.Context(0) as ctx:
        check(kg.solve_k_device(ctx, dH, dS, n, n, nk, dw, dC, n), "solve")
        check(kg.fermi_device(ctx, dw, n, nk, wk, nelec, 0.01, 2.0, occ, res, st), "fermi")
        check(kg.density_device(ctx, dC, n, nk, n, dw, occ, wk, 2.0, rho, E), "density")
        torch.cuda.synchronize()
    assert int(st.cpu().numpy()[0]) == 0
    mu, eb, cnt = res.cpu().numpy()
    assert abs(cnt - nelec) <= 1e-9 * nelec
    # all k share S only through the trace identity per k, so check one k at a
    # time: rebuild rho_k from the device C_k and compare with the sum
    C = host(dC)
    w = dw.cpu().numpy()
    f = occ.cpu().numpy()
    r = rho.cpu().numpy().T
    e = E.cpu().numpy().T
    low = np.tril(np.ones((n, n), dtype=bool))
    tr_n = 0.0
    tr_e = 0.0
    for k in range(nk):
        Ck = C[k]
        tr_n += (1.0 / nk) * 2.0 * np.trace((Ck * f[k]) @ Ck.conj().T @ Ss[k]).real
        tr_e += (1.0 / nk) * 2.0 * np.trace((Ck * (f[k] * w[k])) @ Ck.conj().T @ Ss[k]).real
    assert abs(tr_n - cnt) <= 1e-10 * nelec
    assert abs(tr_e - eb) <= 1e-10 * max(1.0, abs(eb)) * n
    # and the device matrices are that same sum (lower triangles)
    rr = sum((1.0 / nk) * 2.0 * (C[k] * f[k]) @ C[k].conj().T for k in range(nk))
    assert np.abs(r - rr)[low].max() <= 1e-12 * np.abs(rr).max()
    ee = sum((1.0 / nk) * 2.0 * (C[k] * (f[k] * w[k])) @ C[k].conj().T for k in range(nk))
    assert np.abs(e - ee)[low].max() <= 1e-12 * np.abs(ee).max()


def test_density_sampled_entries_full_size():
    # the bench workload's size: n = 2000, 16 k-points, half of the states
    # occupied columns; sampled entries against the oracle one by one
    rng = np.random.default_rng(31)
    nk, n, nocc = 16, 2000, 1000
    Ccol = (rng.standard_normal((nk, n, n)) + 1j * rng.standard_normal((nk, n, n))) / np.sqrt(n)
    w = np.sort(rng.standard_normal((nk, n)), axis=1)
    occ = rng.uniform(0, 1, (nk, n))
    wk = np.full(nk, 1.0 / nk)
    r, e, _ = gpu_density(Ccol, w, occ, wk, 2.0, nocc)
    pairs = [(0, 0), (1999, 0), (1999, 1999), (1000, 999), (64, 63), (1234, 17), (700, 700), (1999, 1998)]
    r0, e0 = O.density_entries(Ccol, w, occ, wk, 2.0, pairs, nocc=nocc)
    A = np.abs(Ccol[:, :nocc, :])            # [k, j, i]
    f = wk[:, None] * occ[:, :nocc]
    for q, (a, b) in enumerate(pairs):
        tr = 2.0 * float((A[:, :, a] * A[:, :, b] * f).sum())
        te = 2.0 * float((A[:, :, a] * A[:, :, b] * f * np.abs(w[:, :nocc])).sum())
        assert abs(r[a, b] - r0[q]) <= 8 * nk * nocc * U * tr
        assert abs(e[a, b] - e0[q]) <= 8 * nk * nocc * U * te
