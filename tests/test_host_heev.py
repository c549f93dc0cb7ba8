"""The host's Hermitian eigensolver against numpy: values, residuals and
orthonormality.  Tolerance: Jacobi's n sweeps-worth of backward-stable
rotations, 16 n eps of the largest entry (of 1 for the vectors), eps = 2.2e-16."""

import numpy as np
import pytest

import paper_1708_09689_amd as pv


def matrix(kind, n):
    g = np.random.default_rng(n)
    Z = g.standard_normal((n, n)) + 1j * g.standard_normal((n, n))
    if kind == "random":
        return Z + Z.conj().T
    if kind == "graded":
        d = 10.0 ** -np.linspace(0, 12, n)
        return (Z + Z.conj().T) * np.sqrt(np.outer(d, d))
    if kind == "pairs":
        Q, _ = np.linalg.qr(Z)
        H = (Q * np.repeat(g.standard_normal((n + 1) // 2), 2)[:n]) @ Q.conj().T
        return 0.5 * (H + H.conj().T)
    return np.diag(g.standard_normal(n)).astype(complex) if kind == "diagonal" else np.zeros((n, n), complex)


@pytest.mark.parametrize("kind", ["random", "graded", "pairs", "diagonal", "zero"])
@pytest.mark.parametrize("n", [1, 2, 3, 17, 64, 65])
def test_eigenpairs(kind, n):
    A = matrix(kind, n)
    w, V = pv.pv_host_heev(A)
    w, V = np.asarray(w), np.asarray(V)
    tol = 16 * n * 2.2e-16
    size = np.abs(A).max()
    assert np.all(np.diff(w) >= 0)
    assert np.abs(w - np.linalg.eigvalsh(A)).max() <= tol * n ** 0.5 * size
    assert np.abs(A @ V - V * w).max() <= tol * n ** 0.5 * size
    assert np.abs(V.conj().T @ V - np.eye(n)).max() <= tol
