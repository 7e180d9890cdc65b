"""GPU complex matrix product (the ZGEMMs of Parts 3-4) against the oracle's
plain triple loop, element by element, on ragged sizes spanning several
tiles.  Bound: |fl(AB) - AB| <= c k eps (|A||B|) entrywise."""
import numpy as np
import pytest
import torch

import oracle as O
from gpu_helpers import DEV, EPS, K, check

pytestmark = pytest.mark.gpu


def rnd(rng, *shape):
    return rng.standard_normal(shape) + 1j * rng.standard_normal(shape)


@pytest.mark.parametrize("ta,tb", [("N", "N"), ("C", "N"), ("N", "C"), ("C", "C")])
@pytest.mark.parametrize("m,n,k", [(1, 1, 1), (67, 45, 33), (130, 70, 129), (64, 64, 16)])
def test_zgemm_matches_triple_loop(ta, tb, m, n, k):
    kg = K()
    rng = np.random.default_rng(m * 1000 + n * 10 + k)
    batch = 3
    A = [rnd(rng, m, k) if ta == "N" else rnd(rng, k, m) for _ in range(batch)]
    B = [rnd(rng, k, n) if tb == "N" else rnd(rng, n, k) for _ in range(batch)]
    C0 = [rnd(rng, m, n) for _ in range(batch)]
    alpha, beta = 0.75 - 0.5j, -0.25 + 1j
    to = lambda Ms: torch.from_numpy(np.ascontiguousarray(np.swapaxes(np.array(Ms), -1, -2))).to(DEV)
    dA, dB, dC = to(A), to(B), to(C0)
    lda, ldb = A[0].shape[0], B[0].shape[0]
    with kg.Context(0) as ctx:
        check(kg.zgemm_device(ctx, ta, tb, m, n, k, alpha, dA, lda, A[0].size, dB, ldb, B[0].size, beta,
                              dC, m, m * n, batch))
        torch.cuda.synchronize()
    got = np.swapaxes(dC.cpu().numpy(), -1, -2)
    for q in range(batch):
        ref = O.zgemm(ta, tb, A[q], B[q], alpha=alpha, beta=beta, C=C0[q])
        opA = A[q] if ta == "N" else A[q].conj().T
        opB = B[q] if tb == "N" else B[q].conj().T
        bound = 8 * k * EPS * (abs(alpha) * np.abs(opA) @ np.abs(opB) + abs(beta) * np.abs(C0[q])) + 1e-300
        assert np.all(np.abs(got[q] - ref) <= bound), f"batch {q}: max err {np.abs(got[q]-ref).max()}"


def test_zgemm_lower_only_writes_lower():
    kg = K()
    rng = np.random.default_rng(5)
    n, k = 97, 40
    X = rnd(rng, k, n)
    G = rnd(rng, k, n)
    sentinel = 123.0 + 456.0j
    dX = torch.from_numpy(np.ascontiguousarray(X.T)).to(DEV)
    dG = torch.from_numpy(np.ascontiguousarray(G.T)).to(DEV)
    dC = torch.full((n, n), sentinel, dtype=torch.complex128, device=DEV)
    with kg.Context(0) as ctx:
        check(kg.zgemm_device(ctx, "C", "N", n, n, k, 1.0, dX, k, 0, dG, k, 0, 0.0, dC, n, 0, 1, lower=True))
        torch.cuda.synchronize()
    got = dC.cpu().numpy().T
    ref = X.conj().T @ G
    low = np.tril(np.ones((n, n), dtype=bool))
    assert np.abs(got[low] - ref[low]).max() <= 1e-12 * np.abs(ref).max()
    assert np.all(got[~low] == sentinel)


def test_zgemm_beta_zero_ignores_nan_in_c():
    kg = K()
    rng = np.random.default_rng(6)
    A = rnd(rng, 20, 20)
    dA = torch.from_numpy(np.ascontiguousarray(A.T)).to(DEV)
    dC = torch.full((20, 20), float("nan"), dtype=torch.complex128, device=DEV)
    with kg.Context(0) as ctx:
        check(kg.zgemm_device(ctx, "N", "N", 20, 20, 20, 1.0, dA, 20, 0, dA, 20, 0, 0.0, dC, 20, 0, 1))
        torch.cuda.synchronize()
    assert np.allclose(dC.cpu().numpy().T, A @ A, atol=1e-12)


# the loads straight to LDS at the edges of their steps (8 and 16 of the inner
# dimension) and tiles, with 32 x 32 tiles (one product) and 64 x 64 tiles (a
# batch that fills the chip); operands on 8-byte boundaries only take the
# kernel without those loads and give the same bits
@pytest.mark.parametrize("ta", ["N", "C"])
@pytest.mark.parametrize("tb", ["N", "C"])
@pytest.mark.parametrize("m,n,k,batch", [(1, 1, 1, 1), (33, 31, 7, 1), (64, 65, 8, 1), (40, 70, 17, 2), (65, 64, 9, 130),
                                         (31, 63, 16, 260), (70, 5, 25, 130), (64, 64, 33, 256)])
def test_zgemm_loads_to_lds(ta, tb, m, n, k, batch):
    kg = K()
    g = torch.Generator(device=DEV)
    g.manual_seed(m + 10 * n + 100 * k)

    def ops(shift):
        """Column-major operands, `shift` doubles off a 16-byte boundary."""
        out = []
        for x in (a, b, c):
            buf = torch.empty(x.numel() * 2 + 2, dtype=torch.float64, device=DEV)
            buf[shift:shift + x.numel() * 2] = torch.view_as_real(x).reshape(-1)
            out.append(buf[shift:])
        return out

    a = torch.randn((batch, k, m) if ta == "N" else (batch, m, k), dtype=torch.complex128, device=DEV, generator=g)
    b = torch.randn((batch, n, k) if tb == "N" else (batch, k, n), dtype=torch.complex128, device=DEV, generator=g)
    c = torch.randn((batch, n, m), dtype=torch.complex128, device=DEV, generator=g)
    got = []
    with kg.Context(0) as ctx:
        for shift in (0, 1):
            da, db, dc = ops(shift)
            check(kg.zgemm_device(ctx, ta, tb, m, n, k, 0.75 - 0.5j, da, a.shape[-1], m * k, db, b.shape[-1], n * k,
                                  0.25 + 1.0j, dc, m, m * n, batch), "zgemm")
            torch.cuda.synchronize()
            got.append(torch.view_as_complex(dc[:2 * c.numel()].clone().reshape(batch, n, m, 2)))
    assert torch.equal(torch.view_as_real(got[0]), torch.view_as_real(got[1]))
    A, B, C = (x.cpu().numpy().swapaxes(-1, -2) for x in (a, b, c))
    A = A if ta == "N" else A.conj().swapaxes(-1, -2)
    B = B if tb == "N" else B.conj().swapaxes(-1, -2)
    ref = (0.75 - 0.5j) * (A @ B) + (0.25 + 1.0j) * C
    bound = 8 * k * EPS * (abs(0.75 - 0.5j) * (np.abs(A) @ np.abs(B)) + abs(0.25 + 1.0j) * np.abs(C))
    assert np.all(np.abs(got[0].cpu().numpy().swapaxes(-1, -2) - ref) <= 2 * bound)


# which kernel takes a product: at the edges of two steps of the inner dimension
# (32 for 32 x 32 tiles, 16 for 64 x 64) with and without C read, fewer and more than
# 512 workgroups of 32 x 32 tiles, and 64 x 64 tiles, against the products of
# operands on 8-byte boundaries, which have one kernel
@pytest.mark.parametrize("beta", [0.0, 0.25 + 1.0j])
@pytest.mark.parametrize("m,n,batch", [(70, 33, 2), (97, 65, 60), (65, 64, 130)])
@pytest.mark.parametrize("k", [1, 7, 8, 9, 15, 16, 17, 31, 32, 33, 34])
def test_zgemm_small_inner_dimension(m, n, batch, k, beta):
    kg = K()
    g = torch.Generator(device=DEV)
    g.manual_seed(m + 100 * k)
    a, b, c = (torch.randn(s, dtype=torch.complex128, device=DEV, generator=g)
               for s in ((batch, k, m), (batch, k, n), (batch, n, m)))
    got = []
    with kg.Context(0) as ctx:
        for shift in (0, 1):
            ops = []
            for x in (a, b, c):
                buf = torch.empty(x.numel() * 2 + 2, dtype=torch.float64, device=DEV)
                buf[shift:shift + x.numel() * 2] = torch.view_as_real(x).reshape(-1)
                ops.append(buf[shift:])
            da, db, dc = ops
            check(kg.zgemm_device(ctx, "N", "C", m, n, k, 0.75 - 0.5j, da, m, m * k, db, n, n * k, beta, dc, m, m * n,
                                  batch), "zgemm")
            torch.cuda.synchronize()
            got.append(dc[:2 * c.numel()].clone())
    assert torch.equal(got[0], got[1])
    A, B, C = (x.cpu().numpy().swapaxes(-1, -2) for x in (a, b, c))
    ref = (0.75 - 0.5j) * (A @ B.conj().swapaxes(-1, -2)) + beta * C
    bound = 8 * k * EPS * (abs(0.75 - 0.5j) * (np.abs(A) @ np.abs(B).swapaxes(-1, -2)) + abs(beta) * np.abs(C))
    out = torch.view_as_complex(got[0].reshape(batch, n, m, 2)).cpu().numpy().swapaxes(-1, -2)
    assert np.all(np.abs(out - ref) <= 2 * bound)
