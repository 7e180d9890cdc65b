"""The library's search for the chemical potential, on the host: in a gap it
ends where bisection of the whole bracket ends, at no more than a fifth above its
evaluations (the steps that find out that the slope doesn't fix mu); where the
slope does, with far fewer and at the same root to the rounding of the count."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
G = 2.0


@pytest.fixture(scope="module")
def search(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("fermi") / "fermi_harness.so")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
                           "-I", os.path.join(HERE, "..", "paper_1402_4247_amd", "csrc"),
                           os.path.join(HERE, "fermi_harness.cpp"), "-o", so])
    f = ctypes.CDLL(so).fh_search
    f.restype = ctypes.c_double
    f.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int, ctypes.c_int, ctypes.c_double, ctypes.c_double,
                  ctypes.c_double, ctypes.c_int, ctypes.c_int, ctypes.c_void_p]

    def call(w, wk, nelec, kT, plain=False, rising=True):
        w, wk = np.ascontiguousarray(w), np.ascontiguousarray(wk, dtype=np.float64)
        evals = ctypes.c_int()
        mu = f(w.ctypes.data, wk.ctypes.data, w.shape[1], w.shape[0], nelec, kT, G, rising, plain,
               ctypes.byref(evals))
        return mu, evals.value

    return call


def spectrum(kind, n, nk, rng):
    low = np.arange(n) < n // 2
    bands = np.where(low, -1.0, 1.0) * rng.uniform(0, 2, (nk, n))
    if kind == "gap":
        w = bands + np.where(low, -0.9, 0.9)
    elif kind == "small gap":
        w = bands + np.where(low, -0.3, 0.3)
    elif kind == "core states and a gap":
        w = np.where(np.arange(n) < n // 4, -20 + 0.1 * bands, bands + np.where(low, -0.4, 0.4))
    elif kind == "gap far from zero":
        w = bands + np.where(low, 7.0, 8.6)
    elif kind == "metal":
        w = rng.standard_normal((nk, n))
    else:
        assert kind == "core states and a metal"
        w = np.where(np.arange(n) < n // 4, -20 + 0.1 * bands, rng.standard_normal((nk, n)))
    return np.sort(w, axis=1)


GAPS = ["gap", "small gap", "core states and a gap", "gap far from zero"]


@pytest.mark.parametrize("n,nk", [(40, 1), (130, 3), (333, 2)])
@pytest.mark.parametrize("kT", [1e-4, 0.002, 0.01, 0.02])
@pytest.mark.parametrize("kind", GAPS)
def test_gap(search, kind, kT, n, nk):
    w = spectrum(kind, n, nk, np.random.default_rng(n))
    wk = np.full(nk, 1.0 / nk)
    mu0, plain = search(w, wk, G * (n // 2), kT, plain=True)
    mu, evals = search(w, wk, G * (n // 2), kT)
    assert mu == mu0
    assert evals <= 1.2 * plain, (evals, plain)


@pytest.mark.parametrize("n,nk", [(130, 3), (333, 2)])
@pytest.mark.parametrize("kT", [0.01, 0.02, 0.1])
@pytest.mark.parametrize("kind", ["metal", "core states and a metal"])
def test_metal(search, kind, kT, n, nk):
    rng = np.random.default_rng(n)
    w = spectrum(kind, n, nk, rng)
    wk = rng.uniform(0.5, 1.5, nk)
    wk /= wk.sum()
    nelec = 1.13 * n
    mu0, plain = search(w, wk, nelec, kT, plain=True)
    mu, evals = search(w, wk, nelec, kT)
    f = 1.0 / (1.0 + np.exp((w - mu0) / kT))
    slope = G * float((wk[:, None] * f * (1 - f)).sum()) / kT
    assert abs(mu - mu0) <= 1e-13 * nelec / slope + 4 * np.finfo(float).eps * max(1.0, abs(mu0))
    assert evals <= 0.6 * plain, (evals, plain)


@pytest.mark.parametrize("kind", GAPS + ["metal"])
def test_negative_weights_are_plain_bisection(search, kind):
    # the count may fall then: nothing is concluded from one point to another
    w = spectrum(kind, 60, 3, np.random.default_rng(5))
    wk = np.array([0.7, -0.1, 0.4])
    assert search(w, wk, 60.0, 0.01, rising=False) == search(w, wk, 60.0, 0.01, plain=True)
