"""The Krylov check's square root T^{1/2} e_1 on given matrices, by the
quadrature and by QL, against an eigen-decomposition (eigenvalues below 0
taken as 0).

Bar: both sides are exact for a matrix within E = 8 n^(3/2) eps B of T (B its
Gershgorin bound), which moves the root by at most 2 sqrt(E), and by E / (2
sqrt(mu)) where every eigenvalue is at least mu from 0, as divided differences
of sqrt(max(x, 0)) are at most 1 / (2 sqrt(mu)) there.
"""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

EPS = 2.0**-52


def root(lib, d, e, force_ql=False):
    """(path, s): path 1 by the quadrature, 0 by QL, -1 not found."""
    f = lib.load().pse_internal_tridiag_root
    dp = ctypes.POINTER(ctypes.c_double)
    f.argtypes, f.restype = [ctypes.c_int, ctypes.c_int, dp, dp, dp], ctypes.c_int
    d, e = np.ascontiguousarray(d, float), np.append(np.asarray(e, float), 0.0)
    s = np.empty(len(d))
    path = f(int(force_ql), len(d), d.ctypes.data_as(dp), e.ctypes.data_as(dp), s.ctypes.data_as(dp))
    return path, s


def verify(lib, d, e, label, scale=0):
    """Both paths on 2^(2 scale) T, and the path taken by the spectrum."""
    d, e = np.asarray(d, float), np.asarray(e, float)
    n = len(d)
    lam, q = np.linalg.eigh(np.diag(d) + np.diag(e, 1) + np.diag(e, -1))
    ref = q @ (np.sqrt(np.maximum(lam, 0.0)) * q[0])
    a = np.abs(e)
    bound = float(np.max(np.abs(d) + np.append(a, 0.0) + np.append(0.0, a)))
    E = 8 * n**1.5 * EPS * bound
    mu = float(np.min(np.abs(lam)))
    bar = 2 * np.sqrt(E)
    if mu > 2 * E:
        bar = min(bar, E / (2 * np.sqrt(mu - E)))
    ex = int(np.frexp(bound)[1])  # the power of two T is scaled by, made even
    low = 1e-13 * 2.0 ** (ex + (ex & 1))
    for force in (False, True):
        path, s = root(lib, d * 4.0**scale, e * 4.0**scale, force)
        err = float(np.linalg.norm(s * 0.5**scale - ref))
        print(f"{label} n={n} scale 4^{scale}: smallest eigenvalue {lam[0]:.2e} of bound {bound:.2e}, path {path}, "
              f"err {err:.2e} (bar {bar:.2e})", flush=True)
        assert path in (0, 1)
        if force or n == 1 or lam[0] < low - E:  # (one row: a square root, no quadrature)
            assert path == 0
        elif lam[0] > low + E:
            assert path == 1
        assert err <= bar, label


def tridiagonal(lam, seed):
    """T with the spectrum lam (Householder reduction of Q diag(lam) Q^T)."""
    from scipy.linalg import hessenberg, qr

    n = len(lam)
    q, _ = qr(np.random.default_rng(seed).standard_normal((n, n)))
    h = hessenberg((q * lam) @ q.T)
    return np.diag(h).copy(), np.diag(h, -1).copy()


@pytest.mark.parametrize("n", [2, 3, 5, 17, 63, 64])
@pytest.mark.parametrize("low", [0.3, 1e-6, 3e-13, 1e-14, 1e-15, -1e-15, -1e-6, -0.4])
def test_root_by_spectrum(gpu_lib, n, low):
    """Positive definite from well conditioned to singular, and indefinite."""
    lam = np.linspace(abs(low), 1.0, n)
    lam[0] = low
    d, e = tridiagonal(lam, 100 + n)
    for scale in (-150, 0, 150):
        verify(gpu_lib, d, e, f"low {low:g}", scale)


@pytest.mark.parametrize("sign", [1.0, -1.0])
@pytest.mark.parametrize("n", [1, 2, 4, 64])
def test_root_of_decoupled_rows(gpu_lib, n, sign):
    """Off-diagonal entries that are exactly 0, all or every other one."""
    d = sign * np.linspace(0.5, 1.5, n)
    e = np.zeros(n - 1)
    verify(gpu_lib, d, e, "diagonal")
    e[::2] = 0.25
    verify(gpu_lib, d, e, "pairs")
    verify(gpu_lib, np.zeros(n), np.zeros(n - 1) if n < 2 else e, "zero diagonal")


def test_root_just_below_zero(gpu_lib):
    """Smallest eigenvalues a few roundings below 0, where T shifted by the
    quadrature's smallest nodes is nearly singular."""
    for k in range(0, 41):
        verify(gpu_lib, [1.0, 1.0], [1.0 + k * EPS], f"1 - e = -{k} eps")


def test_root_not_finite(gpu_lib):
    for bad in (np.nan, np.inf):
        for n in (1, 5):
            d, e = np.linspace(1.0, 2.0, n), np.full(n - 1, 0.2)
            d[n // 2] = bad
            path, s = root(gpu_lib, d, e)
            assert path == -1 or not np.all(np.isfinite(s))
