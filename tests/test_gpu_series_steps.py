"""GPU parity of Chebyshev series whose steps touch the accumulator every third
time (for their own term and the two before it): every remainder of the number
of steps, the direct and the staged kernel, generated kernels, out of place, in
place over the input (propagation) and with every step kept (its adjoint).

Tolerances: complex128 1e-12 of the largest entry (the parity bound of series);
complex64 K + 1 steps of 24 roundings at eps = 6e-8, unit coefficients over
sqrt(K + 1): 24 * (K + 1) * eps, below 2e-5 for K <= 9."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1708_09689_amd as pv  # noqa: E402
from oracle import chebtp  # noqa: E402
import workloads as W  # noqa: E402

from gpu_common import Case, dev, host, rel_err  # noqa: E402
from test_gpu_codegen import GenCase  # noqa: E402

A, B = 9.0, 0.1


def series(H, X, coef):
    w0 = X.astype(np.complex128)
    acc = coef[0] * w0
    w1 = (H @ w0 - B * w0) / A
    for k in range(1, len(coef)):
        acc = acc + coef[k] * w1
        w0, w1 = w1, 2.0 * (H @ w1 - B * w1) / A - w0
    return acc


def coefficients(K):
    g = np.random.default_rng(K)
    return (g.standard_normal(K + 1) + 1j * g.standard_normal(K + 1)) / np.sqrt(K + 1.0)


@pytest.mark.parametrize("name,L,per,nb", [("ti", (9, 7, 5), (1, 1, 0), 4), ("weyl", (12, 6, 5), (0, 1, 1), 8),
                                           ("graphene4", (21, 9), (1, 0), 8), ("xz", (11, 4, 6), (1, 0, 1), 4)])
@pytest.mark.parametrize("kernel", [1, 2])
@pytest.mark.parametrize("K", range(1, 10))
@pytest.mark.parametrize("dtype", [np.complex128, np.complex64])
def test_series_of_every_remainder(name, L, per, nb, kernel, K, dtype):
    c128 = dtype == np.complex128
    c = (GenCase if name == "xz" else Case)(name, L, per, seed=61, vdtype=np.float64 if c128 else np.float32)
    pv.pv_lattice_set_tuning(c.lat, pv.PV_C128 if c128 else pv.PV_C64, nb, {"kernel": kernel})
    xh = W.gaussian_block(c.H.shape[0], nb, W.generator(62, K), dtype)
    x, y = dev(xh), dev(np.full_like(xh, np.nan))
    coef = coefficients(K)
    pv.pv_cheb_series(c.lat, x, y, A, B, coef)
    assert rel_err(host(y), series(c.H, xh, coef)) < (1e-12 if c128 else 2e-5)
    assert np.array_equal(host(x), xh)


@pytest.mark.parametrize("M", range(1, 8))
@pytest.mark.parametrize("kernel", [1, 2])
def test_propagation_in_place(M, kernel):
    """Two time steps in place over the packet."""
    c = Case("ti", (9, 7, 5), (1, 1, 0), seed=63)
    pv.pv_lattice_set_tuning(c.lat, pv.PV_C128, 4, {"kernel": kernel})
    x = c.block(4)
    psi = dev(x)
    pv.pv_cheb_propagate(c.lat, psi, A, B, 0.05, M, 2)
    assert rel_err(host(psi), chebtp.propagate(c.H, x, A, B, 0.05, M, 2)) < 1e-12
