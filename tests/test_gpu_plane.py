"""GPU parity of the several-steps-per-pass kernels of 2D lattices against the
explicit matrix: tile edges (a wave owns 64 / nb sites less a halo of the
pass's steps on both sides), walks of one row to many, open and periodic
boundaries, remainders of the steps per pass, stored and absent fields.

Tolerances: complex128 -- the parity bound of the single sweeps, 1e-12 of the
largest entry (moments: absolute, mu_0 = 1).  complex64 -- K steps of at most
a dozen roundings each, eps = 6e-8, at unit norm: K * 12 * eps of the largest
entry."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1708_09689_amd as pv  # noqa: E402
from oracle import kpm  # noqa: E402

from gpu_common import Case, dev, host, rel_err  # noqa: E402

A = {"graphene2": 4.0, "graphene4": 4.0}


def series(H, X, coef, a, b):
    w0 = X.astype(np.complex128)
    w1 = (H @ w0 - b * w0) / a
    acc = coef[0] * w0 + coef[1] * w1
    for c in coef[2:]:
        w0, w1 = w1, 2.0 * (H @ w1 - b * w1) / a - w0
        acc = acc + c * w1
    return acc


def coefficients(K):
    g = np.random.default_rng(K)
    return (g.standard_normal(K + 1) + 1j * g.standard_normal(K + 1)) / np.sqrt(K + 1.0)


SHAPES = [
    ("graphene2", (1, 8), (1, 1), 1), ("graphene2", (3, 9), (0, 1), 1), ("graphene2", (52, 8), (1, 1), 1),
    ("graphene2", (53, 13), (0, 0), 1), ("graphene2", (56, 31), (1, 0), 1), ("graphene2", (57, 300), (0, 1), 1),
    ("graphene2", (430, 70), (0, 0), 1), ("graphene2", (24, 17), (0, 1), 2), ("graphene2", (49, 40), (1, 0), 2),
    ("graphene2", (9, 33), (0, 0), 4), ("graphene2", (100, 9), (1, 1), 4),
    ("graphene4", (2, 8), (1, 1), 1), ("graphene4", (58, 11), (0, 0), 1), ("graphene4", (59, 270), (1, 0), 1),
    ("graphene4", (27, 19), (0, 1), 2), ("graphene4", (21, 10), (1, 1), 4),
    ("graphene4", (117, 143), (0, 1), 1), ("graphene4", (59, 80), (1, 0), 4),
]


@pytest.mark.parametrize("name,L,per,nb", SHAPES)
@pytest.mark.parametrize("K", [2, 6, 7, 12, 17])
def test_series_passes(name, L, per, nb, K):
    c = Case(name, L, per, Wd=0.4, seed=31, with_field=K != 7)
    X = c.block(nb)
    coef = coefficients(K)
    Y = dev(np.zeros_like(X))
    pv.pv_cheb_series(c.lat, dev(X), Y, A[name], 0.1, coef)
    assert rel_err(host(Y), series(c.H, X, coef, A[name], 0.1)) < 1e-12


@pytest.mark.parametrize("name,L,per,nb", SHAPES[3:8] + SHAPES[9:11] + SHAPES[12:])
@pytest.mark.parametrize("vdtype", [np.float32, np.float64])
def test_series_passes_c64(name, L, per, nb, vdtype):
    K = 11
    c = Case(name, L, per, Wd=0.4, seed=32, vdtype=vdtype)
    X = c.block(nb, dtype=np.complex64)
    coef = coefficients(K)
    Y = dev(np.zeros_like(X))
    pv.pv_cheb_series(c.lat, dev(X), Y, A[name], 0.1, coef)
    assert rel_err(host(Y), series(c.H, X, coef, A[name], 0.1)) < K * 12 * 6e-8


@pytest.mark.parametrize("name,L,per,nb", SHAPES)
@pytest.mark.parametrize("M", [4, 14, 26, 128])
def test_moments_passes(name, L, per, nb, M):
    c = Case(name, L, per, Wd=0.4, seed=33)
    r = c.block(nb, kind="phase")
    mu = host(pv.pv_kpm_moments(c.lat, dev(r), M, A[name], 0.0))
    assert np.abs(mu - kpm.moments_doubling(c.H, r, M, A[name], 0.0)).max() < 1e-12


def test_moments_reduced_in_several_parts():
    """More steps than the workspace holds dots for."""
    c = Case("graphene2", (60, 9), (1, 1), Wd=0.4, seed=34)
    r = c.block(1, kind="phase")
    mu = host(pv.pv_kpm_moments(c.lat, dev(r), 300, 4.0, 0.0))
    assert np.abs(mu - kpm.moments_doubling(c.H, r, 300, 4.0, 0.0)).max() < 1e-12


@pytest.mark.parametrize("M", [2, 6, 7, 33])
def test_propagation_in_place_equals_sweeps(M):
    """The propagator in place, in passes and (with a set launch shape) in
    single sweeps; a workspace of the sweeps' size takes the sweeps."""
    c = Case("graphene2", (117, 45), (0, 1), Wd=0.2, seed=35)
    psi = c.block(1)
    a = dev(psi)
    pv.pv_cheb_propagate(c.lat, a, 4.0, 0.1, 1.5, M, 3)
    pv.pv_lattice_set_tuning(c.lat, pv.PV_C128, 1, {"kernel": 1})
    b = dev(psi)
    pv.pv_cheb_propagate(c.lat, b, 4.0, 0.1, 1.5, M, 3)
    assert rel_err(host(a), host(b)) < 1e-12
