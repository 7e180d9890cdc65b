"""Stage parity on the GPU: Householder tridiagonalisation (Procedures 1-6),
the divide-and-conquer tridiagonal eigensolver and the back-transformation
("rearrangement of eigenvectors"), each against the oracle on the same
seeded inputs, at sizes spanning several 64-row tiles and 32-column panels
with ragged tails."""
import numpy as np
import pytest
import torch

import oracle as O
from gpu_helpers import DEV, EPS, K, check, dev, host

pytestmark = pytest.mark.gpu


def mx(a):
    a = np.asarray(a)
    return float(np.abs(a).max()) if a.size else 0.0


def rand_herm(rng, n):
    A = rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))
    return (A + A.conj().T) / 2


def gpu_hetrd(As, nb=0):
    kg = K()
    nk, n = As.shape[0], As.shape[1]
    dA = dev(As)
    dd = torch.zeros((nk, n), dtype=torch.float64, device=DEV)
    de = torch.zeros((nk, n), dtype=torch.float64, device=DEV)
    dtau = torch.zeros((nk, n), dtype=torch.complex128, device=DEV)
    dV = torch.zeros((nk, n, n), dtype=torch.complex128, device=DEV)
    with kg.Context(0) as ctx:
        check(kg.hetrd_device(ctx, dA, n, n, nk, dd, de, dtau, dV, opts=kg.make_opts(panel_nb=nb)), "hetrd")
        torch.cuda.synchronize()
    return dd.cpu().numpy(), de.cpu().numpy(), dtau.cpu().numpy(), host(dV)


# n <= 128 runs in one launch with the matrix in registers; with nb = 0 orders up to
# 160 hand over to it at the first panel start whose trailing order is at most 128,
# and larger ones to a group of workgroups, these whole; with a width given, all
# hand over at 128
@pytest.mark.parametrize("n,nb", [(1, 0), (2, 0), (3, 0), (17, 0), (64, 0), (65, 0), (128, 0), (129, 0), (130, 0),
                                  (161, 0), (200, 0), (200, 8), (97, 64), (250, 24), (300, 48)])
def test_hetrd_matches_oracle(n, nb):
    rng = np.random.default_rng(n + 7 * nb)
    nk = 2
    As = np.stack([rand_herm(rng, n) for _ in range(nk)])
    d, e, tau, V = gpu_hetrd(As, nb)
    for q in range(nk):
        A = As[q]
        nf = np.linalg.norm(A)
        d0, e0, tau0, V0 = O.zhetrd(A)
        tol = 64 * n * EPS * nf
        assert mx(d[q] - d0) <= tol, f"d k={q}: {mx(d[q]-d0)}"
        assert mx(e[q, : n - 1] - e0) <= tol, f"e k={q}: {mx(e[q, : n - 1] - e0)}"
        # same reflector convention -> same tau and v up to rounding
        assert mx(tau[q, : n - 1] - tau0) <= 64 * n * EPS * 4, f"tau: {mx(tau[q, : n - 1] - tau0)}"
        assert mx(V[q] - V0) <= 64 * n * EPS * 16, f"V: {mx(V[q] - V0)}"
        # similarity: spectrum of the GPU T equals that of A
        wg = O.bisect_eigs(d[q], e[q, : n - 1])
        assert mx(wg - np.sort(np.linalg.eigvalsh(A))) <= tol


def gpu_stedc(ds, es):
    kg = K()
    nk, n = ds.shape
    dd = torch.from_numpy(np.ascontiguousarray(ds)).to(DEV)
    de = torch.zeros((nk, n), dtype=torch.float64, device=DEV)
    de[:, : n - 1] = torch.from_numpy(np.ascontiguousarray(es)).to(DEV)
    dw = torch.zeros((nk, n), dtype=torch.float64, device=DEV)
    dZ = torch.zeros((nk, n, n), dtype=torch.float64, device=DEV)
    st = torch.zeros(nk, dtype=torch.int32, device=DEV)
    with kg.Context(0) as ctx:
        check(kg.stedc_device(ctx, dd, de, n, nk, dw, dZ, st), "stedc")
        torch.cuda.synchronize()
    return dw.cpu().numpy(), np.swapaxes(dZ.cpu().numpy(), -1, -2), st.cpu().numpy()


def tri(d, e):
    return np.diag(d) + np.diag(e, 1) + np.diag(e, -1)


def stedc_cases():
    rng = np.random.default_rng(42)
    out = []
    for n in [1, 2, 3, 5, 33, 64, 100, 257, 600]:
        out.append((f"rand{n}", rng.standard_normal(n), rng.standard_normal(max(n - 1, 0))))
    n = 50
    out.append(("toeplitz", np.full(n, 0.3), np.full(n - 1, -1.7)))
    n = 60
    out.append(("clement", np.zeros(n), np.sqrt(np.arange(1, n) * (n - np.arange(1, n)))))
    n = 21
    out.append(("wilkinson21", np.abs(np.arange(n) - 10.0), np.ones(n - 1)))
    n = 40
    out.append(("diagonal", rng.standard_normal(n), np.zeros(n - 1)))
    n = 64
    out.append(("glued", np.ones(n), np.concatenate([np.full(31, 1e-9), [0.5], np.full(31, 1e-9)])))
    n = 45
    out.append(("zero", np.zeros(n), np.zeros(n - 1)))
    return out


@pytest.mark.parametrize("name,d,e", stedc_cases(), ids=lambda x: x if isinstance(x, str) else "")
def test_stedc_matches_oracle(name, d, e):
    n = len(d)
    nk = 2
    ds = np.stack([d, 2.0 * d])
    es = np.stack([e, 2.0 * e]) if n > 1 else np.zeros((nk, 0))
    w, Z, st = gpu_stedc(ds, es.reshape(nk, max(n - 1, 0)))
    assert np.all(st == 0)
    for q in range(nk):
        T = tri(ds[q], es[q]) if n > 1 else np.diag(ds[q])
        w0, Z0 = O.tridiag_ql(ds[q], es[q])
        nt = max(np.abs(T).max(), 1e-300)
        assert np.all(np.diff(w[q]) >= 0)
        assert mx(w[q] - w0) <= 16 * n * EPS * nt, f"w: {mx(w[q] - w0)}"
        assert np.linalg.norm(T @ Z[q] - Z[q] * w[q]) <= 16 * n * EPS * max(np.linalg.norm(T), 1e-300) + 1e-300
        assert mx(Z[q].T @ Z[q] - np.eye(n)) <= 16 * n * EPS, f"orth: {mx(Z[q].T @ Z[q] - np.eye(n))}"
        # vectors of well-separated eigenvalues agree with QL's up to sign
        gaps = np.minimum(np.r_[np.inf, np.diff(w0)], np.r_[np.diff(w0), np.inf]) / nt
        sep = gaps >= 1e-6
        if sep.any():
            ov = np.abs(np.sum(Z[q] * Z0, axis=0))
            assert np.max(1 - ov[sep]) <= 1e-10


@pytest.mark.parametrize("n", [2, 40, 130])
def test_back_transform_matches_oracle(n):
    kg = K()
    rng = np.random.default_rng(900 + n)
    nk = 2
    As = np.stack([rand_herm(rng, n) for _ in range(nk)])
    d, e, tau, V = gpu_hetrd(As)
    Zs = np.stack([np.linalg.qr(rng.standard_normal((n, n)))[0] for _ in range(nk)]).astype(complex)
    dV = dev(V)
    dtau = torch.from_numpy(tau).to(DEV)
    dU = dev(Zs)
    with kg.Context(0) as ctx:
        check(kg.unmtr_device(ctx, dV, dtau, n, nk, dU, n), "unmtr")
        torch.cuda.synchronize()
    U = host(dU)
    for q in range(nk):
        ref = O.apply_q(V[q], tau[q, : n - 1], Zs[q])
        assert np.abs(U[q] - ref).max() <= 32 * n * EPS


@pytest.mark.parametrize("n", [1, 3, 70, 193])
def test_eigen_hh_matches_oracle(n):
    kg = K()
    rng = np.random.default_rng(300 + n)
    nk = 3
    As = np.stack([rand_herm(rng, n) for _ in range(nk)])
    dA = dev(As)
    dw = torch.zeros((nk, n), dtype=torch.float64, device=DEV)
    dY = torch.zeros((nk, n, n), dtype=torch.complex128, device=DEV)
    st = torch.full((nk,), -7, dtype=torch.int32, device=DEV)
    with kg.Context(0) as ctx:
        check(kg.eigh_device(ctx, dA, n, n, nk, dw, dY, st), "eigh")
        torch.cuda.synchronize()
    assert np.all(st.cpu().numpy() == 0)
    w = dw.cpu().numpy()
    Y = host(dY)
    for q in range(nk):
        A = As[q]
        w0, Y0 = O.eigen_hh(A)
        nf = np.linalg.norm(A)
        assert np.abs(w[q] - w0).max() <= 1e-10 * max(np.abs(w0).max(), 1e-300)
        assert np.linalg.norm(A @ Y[q] - Y[q] * w[q]) <= 32 * n * EPS * nf
        assert np.abs(Y[q].conj().T @ Y[q] - np.eye(n)).max() <= 32 * n * EPS


# the triangular factors at the edges of their 16- and 32-column halves and of
# the 64-column blocks, alone, in pairs and left over
@pytest.mark.parametrize("n", [3, 17, 18, 33, 34, 50, 65, 66, 82, 129, 146, 193, 194])
def test_back_transform_block_edges(n):
    test_back_transform_matches_oracle(n)


def gpu_stebz(ds, es):
    kg = K()
    nk, n = ds.shape
    dd = torch.from_numpy(np.ascontiguousarray(ds)).to(DEV)
    de = torch.zeros((nk, n), dtype=torch.float64, device=DEV)
    de[:, : n - 1] = torch.from_numpy(np.ascontiguousarray(es)).to(DEV)
    dw = torch.full((nk, n), np.nan, dtype=torch.float64, device=DEV)
    with kg.Context(0) as ctx:
        check(kg.stebz_device(ctx, dd, de, n, nk, dw), "stebz")
        torch.cuda.synchronize()
    return dw.cpu().numpy()


@pytest.mark.parametrize("name,d,e", stedc_cases(), ids=lambda x: x if isinstance(x, str) else "")
def test_stebz_matches_oracle(name, d, e):
    # eigenvalues only by bisection: against the oracle's QL and its Sturm
    # bisection, within the backward-stable bound of a few eps ||T|| per value
    n = len(d)
    nk = 2
    ds = np.stack([d, -3.0 * d])
    es = np.stack([e, 3.0 * e]) if n > 1 else np.zeros((nk, 0))
    w = gpu_stebz(ds, es.reshape(nk, max(n - 1, 0)))
    for q in range(nk):
        T = tri(ds[q], es[q]) if n > 1 else np.diag(ds[q])
        nt = max(np.abs(T).max(), 1e-300)
        w0, _ = O.tridiag_ql(ds[q], es[q])
        wb = O.bisect_eigs(ds[q], es[q])
        assert np.all(np.diff(w[q]) >= 0)
        # bisection's bound has an absolute term from the pivot floor (the
        # smallest normal number), which is all there is for T = 0
        tol = 8 * n * EPS * nt + 4 * np.finfo(np.float64).tiny
        assert mx(w[q] - w0) <= tol, f"vs QL: {mx(w[q] - w0)}"
        assert mx(w[q] - wb) <= tol, f"vs bisection: {mx(w[q] - wb)}"


def test_stebz_closed_forms():
    # Toeplitz: a + 2 b cos(j pi / (n + 1)); Clement: -(n-1), -(n-3), ..., n-1
    n = 200
    a, b = 0.3, -1.7
    j = np.arange(1, n + 1)
    toe = np.sort(a + 2 * b * np.cos(j * np.pi / (n + 1)))
    m = 151
    cle = np.arange(-(m - 1), m, 2, dtype=float)
    w1 = gpu_stebz(np.full((1, n), a), np.full((1, n - 1), b))[0]
    w2 = gpu_stebz(np.zeros((1, m)), np.sqrt(np.arange(1, m) * (m - np.arange(1, m)))[None])[0]
    assert mx(w1 - toe) <= 8 * EPS * 2 * abs(b) * 4
    assert mx(w2 - cle) <= 16 * EPS * m


# bisection at the edges of its lane counts (64, 16, 8 and 4 lanes for n nk up to
# 1024, 4096, 8192 and beyond) and of T in LDS (4096 rows): Toeplitz matrices,
# each problem with its own shift and scale, tolerance as above
@pytest.mark.parametrize("n,nk", [(1, 3), (2, 2), (63, 1), (1024, 1), (65, 16), (1365, 3), (4096, 1), (4097, 1),
                                  (100, 82), (5, 1700)])
def test_stebz_lane_counts(n, nk):
    a = 0.3 - 0.01 * np.arange(nk)
    b = -1.7 + 0.0005 * np.arange(nk)
    j = np.arange(1, n + 1)
    w = gpu_stebz(np.repeat(a[:, None], n, 1), np.repeat(b[:, None], n - 1, 1))
    ref = np.sort(a[:, None] + 2 * b[:, None] * np.cos(j * np.pi / (n + 1)), axis=1)
    # the shift reaches 17 and is then the scale of the matrix
    assert np.all(np.abs(w - ref).max(axis=1) <= 8 * EPS * 4 * np.maximum(2 * np.abs(b), np.abs(a)))


# the resident reduction at the edges of its tiles (16), of its two tile
# counts (64, 128), at the smallest trailing orders and handed over to with a
# ragged trailing order; tolerances as above
@pytest.mark.parametrize("n", [4, 15, 16, 18, 31, 33, 48, 63, 66, 80, 111, 113, 127, 140])
def test_resident_reduction_edges(n):
    test_hetrd_matches_oracle(n, 0)


# groups of workgroups: orders at the edges of their shapes (256, 384, 512) and
# of their tiles, more problems than run at once, and the panels before the
# hand-over
@pytest.mark.parametrize("n", [161, 175, 256, 257, 272, 385, 520])
def test_group_reduction_matches_oracle(n):
    test_hetrd_matches_oracle(n, 0)


def spectrum_check(n, nk, seed):
    """T and V of nk reductions against the matrices: the spectrum of T, and
    Q^H A Q = T through the reflectors of the first and last problem."""
    rng = np.random.default_rng(seed)
    As = np.stack([rand_herm(rng, n) for _ in range(nk)])
    d, e, tau, V = gpu_hetrd(As)
    for q in sorted({0, nk // 2, nk - 1}):
        tol = 64 * n * EPS * np.linalg.norm(As[q])
        T = np.diag(d[q]) + np.diag(e[q, : n - 1], 1) + np.diag(e[q, : n - 1], -1)
        assert mx(np.linalg.eigvalsh(T) - np.linalg.eigvalsh(As[q])) <= tol
        B = As[q].copy()
        for i in range(n - 1):
            v, t = V[q][:, i], tau[q, i]
            B -= np.outer(np.conj(t) * v, v.conj() @ B)   # H_i^H B, H_i = I - t v v^H
        for i in range(n - 1):
            v, t = V[q][:, i], tau[q, i]
            B -= np.outer(B @ v, t * v.conj())            # ... B H_i
        assert mx(B - T) <= tol


@pytest.mark.parametrize("n,nk", [(200, 70), (500, 20), (640, 1), (641, 2), (768, 3), (900, 2), (1024, 1), (1090, 1)])
def test_group_reduction_spectrum(n, nk):
    spectrum_check(n, nk, 31 * n + nk)


# blocked columns at the edges of the update's batches (16 panel columns, 32
# and 64 per panel) and of its row blocks, down to the resident reduction
@pytest.mark.parametrize("n,nb", [(193, 1), (150, 5), (257, 16), (258, 17), (322, 33), (200, 64)])
def test_blocked_column_edges(n, nb):
    test_hetrd_matches_oracle(n, nb)


def test_group_given_up_is_reduced_in_memory():
    """No member waits for the others: every group is given up and the
    problems are reduced with the matrix in memory, with the same results."""
    import ctypes
    lib = K().lib
    lib.kgev_internal_group_wait.argtypes = [ctypes.c_int64]
    try:
        lib.kgev_internal_group_wait(0)
        test_hetrd_matches_oracle(230, 0)
        spectrum_check(300, 5, 77)
    finally:
        lib.kgev_internal_group_wait(-1)


class GroupHooks:
    """The library's switches for groups that are given up, at their defaults
    afterwards: at once (before they start), or late (the last problem's lacks a
    member, whose columns the others wait for until their looks run out).
    given_up(): the problems reduced in memory so far."""

    def __enter__(self):
        import ctypes
        self.lib = K().lib
        self.lib.kgev_internal_group_wait.argtypes = [ctypes.c_int64]
        self.lib.kgev_internal_group_lacks_one.argtypes = [ctypes.c_int32]
        self.lib.kgev_internal_groups_given_up.restype = ctypes.c_int64
        return self

    def __exit__(self, *exc):
        self.set(None)

    def set(self, how):
        self.lib.kgev_internal_group_lacks_one(1 if how == "late" else 0)
        self.lib.kgev_internal_group_wait(0 if how == "at once" else -1)

    def given_up(self):
        return self.lib.kgev_internal_groups_given_up()


# one and two rows a thread, edges of the tiles, one and several problems, a
# hand-over after blocked columns
@pytest.mark.parametrize("n,nk,how", [(161, 2, "at once"), (200, 3, "at once"), (257, 1, "at once"),
                                      (333, 3, "at once"), (512, 2, "at once"), (513, 1, "at once"),
                                      (640, 2, "at once"), (777, 1, "at once"), (1024, 1, "at once"),
                                      (1090, 2, "at once"), (200, 3, "late"), (600, 1, "late")])
def test_given_up_group_has_the_same_bits(n, nk, how):
    rng = np.random.default_rng(n)
    As = np.stack([rand_herm(rng, n) for _ in range(nk)])
    with GroupHooks() as hooks:
        counts = [hooks.given_up()]
        ref = gpu_hetrd(As)
        counts.append(hooks.given_up())
        hooks.set(how)
        got = gpu_hetrd(As)
        hooks.set(None)
        counts.append(hooks.given_up())
    assert np.diff(counts).tolist() == [0, nk if how == "at once" else 1]
    for name, a, b in zip(("d", "e", "tau", "V"), ref, got):
        assert np.array_equal(a, b), name


@pytest.mark.parametrize("n,nk", [(200, 2), (520, 1)])
def test_given_up_group_has_the_same_bits_mixed(n, nk):
    # the complex64 reduction, through the mixed-precision solve
    kg = K()
    rng = np.random.default_rng(n)
    dH = dev(np.stack([rand_herm(rng, n) for _ in range(nk)]))
    dS = dev(np.stack([np.eye(n) + 0.01 * rand_herm(rng, n) / n for _ in range(nk)]))
    outs = []
    with GroupHooks() as hooks, kg.Context(0) as ctx:
        for how in (None, "at once"):
            w = torch.zeros((nk, n), dtype=torch.float64, device=DEV)
            C = torch.zeros((nk, n, n), dtype=torch.complex128, device=DEV)
            before = hooks.given_up()
            hooks.set(how)
            check(kg.solve_k_device(ctx, dH, dS, n, n, nk, w, C, n, opts=kg.make_opts(precision=kg.PREC_FP32_REFINE)))
            hooks.set(None)
            # S in complex128 and A in complex64
            assert hooks.given_up() - before == (2 * nk if how else 0)
            outs.append((w, C))
    for w, C in outs[1:]:
        assert torch.equal(w, outs[0][0]) and torch.equal(C, outs[0][1])


def test_stream_compute_units():
    import ctypes
    lib = K().lib
    lib.kgev_internal_stream_units.argtypes = [ctypes.c_void_p]
    units = torch.cuda.get_device_properties(0).multi_processor_count
    for handle in (None, 1, 2):          # the null, the legacy and the per-thread stream
        assert lib.kgev_internal_stream_units(handle) == units
    assert lib.kgev_internal_stream_units(torch.cuda.Stream().cuda_stream) == units


# on a partition of the GPU or under a mask: smaller groups after more blocked
# columns, or none, and none that waits for members in vain
@pytest.mark.parametrize("n,nk,units", [(400, 2, 32), (600, 3, 64), (300, 1, 8), (1100, 1, 128)])
def test_fewer_compute_units(n, nk, units):
    lib = K().lib
    with GroupHooks() as hooks:
        before = hooks.given_up()
        try:
            lib.kgev_internal_compute_units(units)
            spectrum_check(n, nk, 13 * n)
        finally:
            lib.kgev_internal_compute_units(0)
        assert hooks.given_up() == before


def shares_of(n, nk):
    """The shapes {(tile rows, tile columns)} that reduce order n whole, and for
    each the most compute units with which it is chosen."""
    import ctypes
    f = K().lib.kgev_internal_hetrd_plan
    f.argtypes = [ctypes.c_int32, ctypes.c_int32, ctypes.c_int64, ctypes.c_int32, ctypes.c_void_p]
    out = {}
    for units in range(256, 0, -1):
        plan = (ctypes.c_int32 * 4)()
        f(n, 32, nk, units, plan)
        if plan[0] == n and plan[3]:
            out.setdefault((plan[1], plan[2]), units)
    return out


# the widths of a member's share, at orders whose last member and last tile are
# short and where they are not: the sums do not depend on the share
@pytest.mark.parametrize("n,nk,shapes", [(200, 3, [(2, 1), (2, 2), (2, 4)]), (256, 1, [(2, 1), (2, 2), (2, 4)]),
                                         (300, 2, [(3, 1), (3, 2), (3, 3)]), (384, 1, [(3, 1), (3, 2), (3, 3)]),
                                         (500, 2, [(4, 1), (4, 2)]), (600, 2, [(5, 1), (5, 2)]),
                                         (640, 1, [(5, 1), (5, 2)])])
def test_group_shares_give_the_same_bits(n, nk, shapes):
    kg = K()
    units = shares_of(n, nk)
    assert set(shapes) <= set(units)
    rng = np.random.default_rng(17 * n)
    As = np.stack([rand_herm(rng, n) for _ in range(nk)])
    dH = dev(As)
    dS = dev(np.stack([np.eye(n) + 0.01 * rand_herm(rng, n) / n for _ in range(nk)]))
    outs = []
    with GroupHooks() as hooks, kg.Context(0) as ctx:
        before = hooks.given_up()
        for shape in shapes:
            try:
                kg.lib.kgev_internal_compute_units(units[shape])
                d, e, tau, V = gpu_hetrd(As)
                # complex64, through the mixed-precision solve
                w = torch.zeros((nk, n), dtype=torch.float64, device=DEV)
                C = torch.zeros((nk, n, n), dtype=torch.complex128, device=DEV)
                check(kg.solve_k_device(ctx, dH, dS, n, n, nk, w, C, n,
                                        opts=kg.make_opts(precision=kg.PREC_FP32_REFINE)))
                torch.cuda.synchronize()
            finally:
                kg.lib.kgev_internal_compute_units(0)
            outs.append((d, e, tau, V, w.cpu().numpy(), C.cpu().numpy()))
        assert hooks.given_up() == before
    for q in range(nk):
        T = np.diag(outs[0][0][q]) + np.diag(outs[0][1][q, : n - 1], 1) + np.diag(outs[0][1][q, : n - 1], -1)
        assert mx(np.linalg.eigvalsh(T) - np.linalg.eigvalsh(As[q])) <= 64 * n * EPS * np.linalg.norm(As[q])
    for shape, out in zip(shapes[1:], outs[1:]):
        for name, a, b in zip(("d", "e", "tau", "V", "mixed w", "mixed C"), outs[0], out):
            assert np.array_equal(a, b), f"{name}: {shape}"


# merges with chains of deflation rotations, long runs of negligible
# components, tiny and graded blocks; the segment sizes about the deflation's
# steps of 256 rows; tolerances as test_stedc_matches_oracle
def merge_cases():
    rng = np.random.default_rng(7)
    out = []
    for n in (15, 16, 17, 32, 255, 256, 257, 513):
        out.append((f"edge{n}", rng.standard_normal(n), rng.standard_normal(n - 1)))
    n = 200
    out.append(("repeated", np.tile([1.0, 2.0, 2.0, 1.0], n // 4), np.where(np.arange(n - 1) % 4 == 3, 1e-9, 0.3)))
    out.append(("nearly-diagonal", rng.standard_normal(n), 1e-13 * rng.standard_normal(n - 1)))
    out.append(("graded", 10.0 ** -np.linspace(0, 40, n), 10.0 ** -np.linspace(0.5, 40.5, n - 1)))
    d, e = rng.standard_normal(n), rng.standard_normal(n - 1)
    d[100:120] *= 1e-180
    e[99:120] *= 1e-180
    out.append(("tiny-block", d, e))
    out.append(("constant", np.full(300, 0.7), np.full(299, 0.25)))
    return out


@pytest.mark.parametrize("name,d,e", merge_cases(), ids=lambda x: x if isinstance(x, str) else "")
def test_stedc_merges(name, d, e):
    test_stedc_matches_oracle(name, d, e)


# the product of a merge takes one half's columns and the mixed ones for rows of
# that half: halves at and off the edges of its 64-row tiles, with deflation
# rotations inside each half and across them
@pytest.mark.parametrize("n", [66, 127, 128, 129, 191, 260, 400])
@pytest.mark.parametrize("coupling", [1.0, 1e-6, 1e-15])
def test_stedc_halves(n, coupling):
    rng = np.random.default_rng(n)
    d = np.tile([1.0, 2.0, 3.0, 3.0], (n + 3) // 4)[:n] + 1e-3 * rng.integers(0, 3, n)
    test_stedc_matches_oracle("halves", d, coupling * rng.uniform(0.1, 0.4, n - 1))


# chains of deflation rotations at the edges of the 64 candidates and 64 starts
# that are read at a time, with the lists in LDS and (n > 2700) in memory: one
# chain over everything, a chain per pair of equal poles (the halves of a Toeplitz
# matrix with an even order have the same spectrum), and many short ones
@pytest.mark.parametrize("kind", ["one chain", "pairs", "short chains"])
@pytest.mark.parametrize("n", [34, 63, 64, 65, 66, 128, 130, 132, 258, 700, 2750])
def test_stedc_chains(n, kind):
    rng = np.random.default_rng(n)
    if kind == "one chain":
        d, e = np.ones(n), np.full(n - 1, 1e-13)
    elif kind == "pairs":
        d, e = np.full(n, 0.3), np.full(n - 1, -1.7)
    else:
        d, e = np.sort(rng.integers(0, n // 4 + 1, n)).astype(float), 1e-15 * rng.standard_normal(n - 1)
    w, Z, st = gpu_stedc(d[None], e[None])
    assert np.all(st == 0)
    nt = max(np.abs(d).max(), np.abs(e).max())
    if kind == "pairs":
        assert mx(w[0] - np.sort(0.3 + 2 * -1.7 * np.cos(np.arange(1, n + 1) * np.pi / (n + 1)))) <= 16 * n * EPS * nt
    Zd = torch.from_numpy(Z[0].copy()).to(DEV)
    TZ = torch.from_numpy(d).to(DEV)[:, None] * Zd
    ed = torch.from_numpy(e).to(DEV)[:, None]
    TZ[1:] += ed * Zd[:-1]
    TZ[:-1] += ed * Zd[1:]
    norm = np.sqrt((d ** 2).sum() + 2 * (e ** 2).sum())
    assert float((TZ - Zd * torch.from_numpy(w[0]).to(DEV)).norm()) <= 16 * n * EPS * norm
    assert float((Zd.T @ Zd - torch.eye(n, dtype=torch.float64, device=DEV)).abs().max()) <= 16 * n * EPS
