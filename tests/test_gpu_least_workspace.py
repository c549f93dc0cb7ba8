"""Workspaces below the size that *_workspace_size() asks for, down to the least
that a call takes: the results of the full size up to rounding (2D lattices run
sweeps instead of passes, moments are reduced in smaller groups), nothing
written past the bytes that were given, and one byte less refused.

Tolerances: complex128, the same recurrence in another order of roundings,
1e-12 at unit norm; complex64 moments of the same FP32 vectors differ by the
order of FP64 sums alone."""

import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1708_09689_amd as pv  # noqa: E402

from gpu_common import MODELS  # noqa: E402

GUARD = 4096


def up(n):
    return (n + 255) // 256 * 256


class Work:
    """A workspace of n bytes with guard bytes behind it."""

    def __init__(self, n):
        self.n = n
        self.t = torch.full((n + GUARD,), 0xA5, dtype=torch.uint8, device="cuda")

    def ptr(self):
        return ctypes.c_void_p(self.t.data_ptr())

    def check(self):
        torch.cuda.synchronize()
        assert bool((self.t[self.n:] == 0xA5).all()), "bytes past the workspace were written"


def stream():
    return ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)


def lattice(name, L, per, dtype=torch.complex128):
    code, params, _ = MODELS[name]
    st = pv.pv_model_stencil(code, params)
    lat = pv.Lattice(L, per, st)
    g = torch.Generator(device="cuda").manual_seed(61)
    n = lat.n_rows if st["pot_mode"] == pv.PV_POT_ORBITAL else lat.n_sites
    lat.set_potential(torch.rand(n, dtype=torch.float64 if dtype == torch.complex128 else torch.float32, device="cuda",
                                 generator=g))
    return lat, g


def start(lat, nb, dtype, g, offset=0):
    buf = torch.randn(lat.n_rows * nb + 2, dtype=torch.complex128, device="cuda", generator=g)
    r = buf[:lat.n_rows * nb].view(lat.n_rows, nb)
    r = (r / torch.linalg.vector_norm(r, dim=0) * lat.n_rows ** 0.5).to(dtype)
    out = torch.empty(lat.n_rows * nb + 2, dtype=dtype, device="cuda")
    v = out[offset:offset + lat.n_rows * nb].view(lat.n_rows, nb)
    v.copy_(r)
    return v


def partial_bytes(lat, nb):
    return pv.lib().pv_spmmv_workspace_size(lat.handle, pv.PV_C128, nb) - up(3 * nb * 8)


@pytest.mark.parametrize("name,L,per,nb,dtype,offset", [
    ("ti", (7, 6, 5), (1, 0, 1), 2, torch.complex128, 0), ("ti", (31, 20, 9), (1, 1, 1), 8, torch.complex64, 0),
    # complex64 off 16 bytes, large enough to be staged: the steps that read r have another launch shape
    ("ti", (65, 64, 64), (1, 1, 0), 1, torch.complex64, 1),
    ("graphene2", (57, 60), (0, 1), 2, torch.complex128, 0), ("graphene4", (70, 33), (1, 0), 1, torch.complex128, 0)])
@pytest.mark.parametrize("M,buffers", [(4, 2), (24, 2), (24, 3), (24, 5), (26, 12), (140, 7), (140, 63), (140, 64)])
def test_moments(name, L, per, nb, dtype, offset, M, buffers):
    lat, g = lattice(name, L, per, dtype)
    code = pv.PV_C128 if dtype == torch.complex128 else pv.PV_C64
    r = start(lat, nb, dtype, g, offset)
    assert (r.data_ptr() % 16 == 0) == (offset == 0)
    vb, pb = up(lat.n_rows * nb * r.element_size()), partial_bytes(lat, nb)
    full = pv.lib().pv_kpm_workspace_size(lat.handle, code, nb, M)
    mus = []
    for n in (full, min(full, 2 * vb + buffers * pb)):
        w = Work(n)
        mu = torch.full((nb, M), float("nan"), dtype=torch.float64, device="cuda")
        st = pv.lib().pv_kpm_moments(lat.handle, code, nb, M, 9.0, 0.1, ctypes.c_void_p(r.data_ptr()),
                                     ctypes.c_void_p(mu.data_ptr()), w.ptr(), n, stream())
        assert st == 0, pv.lib().pv_last_error()
        w.check()
        mus.append(mu)
    assert (mus[0] - mus[1]).abs().max() <= 1e-12
    w = Work(2 * vb + 2 * pb)
    assert pv.lib().pv_kpm_moments(lat.handle, code, nb, M, 9.0, 0.1, ctypes.c_void_p(r.data_ptr()),
                                   ctypes.c_void_p(mu.data_ptr()), w.ptr(), w.n - 1, stream()) == 4


@pytest.mark.parametrize("name,L,per,nb", [("graphene2", (57, 60), (0, 1), 2), ("graphene4", (259, 261), (1, 0), 1),
                                           ("ti", (9, 8, 7), (1, 1, 0), 4)])
def test_series_and_propagation(name, L, per, nb):
    lat, g = lattice(name, L, per)
    X = start(lat, nb, torch.complex128, g)
    vb, K = up(lat.n_rows * nb * 16), 23
    coef = np.random.default_rng(5).standard_normal((K + 1, 2)) / np.sqrt(K + 1.0)
    outs = []
    full = pv.lib().pv_cheb_series_workspace_size(lat.handle, pv.PV_C128, nb)
    for n in (full, 3 * vb, 2 * vb):
        w, Y = Work(n), torch.full_like(X, float("nan"))
        st = pv.lib().pv_cheb_series(lat.handle, pv.PV_C128, nb, 9.0, 0.1, K, coef.ctypes.data_as(pv._dp),
                                     ctypes.c_void_p(X.data_ptr()), ctypes.c_void_p(Y.data_ptr()), w.ptr(), n, stream())
        assert st == 0, pv.lib().pv_last_error()
        w.check()
        outs.append(Y)
    assert pv.lib().pv_cheb_series(lat.handle, pv.PV_C128, nb, 9.0, 0.1, K, coef.ctypes.data_as(pv._dp),
                                   ctypes.c_void_p(X.data_ptr()), ctypes.c_void_p(Y.data_ptr()), w.ptr(), 2 * vb - 1,
                                   stream()) == 4
    for Y in outs[1:]:
        assert (Y - outs[0]).abs().max() <= 1e-12 * outs[0].abs().max()
    outs = []
    full = pv.lib().pv_cheb_propagate_workspace_size(lat.handle, pv.PV_C128, nb)
    for n in (full, 4 * vb, 3 * vb):
        w, psi = Work(n), X.clone()
        st = pv.lib().pv_cheb_propagate(lat.handle, pv.PV_C128, nb, 9.0, 0.1, 0.5, 14, 3, ctypes.c_void_p(psi.data_ptr()),
                                        w.ptr(), n, stream())
        assert st == 0, pv.lib().pv_last_error()
        w.check()
        outs.append(psi)
    for psi in outs[1:]:
        assert (psi - outs[0]).abs().max() <= 1e-12 * outs[0].abs().max()


@pytest.mark.parametrize("kernel", [1, 2])
@pytest.mark.parametrize("M", [6, 50])
def test_batch(kernel, M):
    """The batch's buffers of partial dots come last: a workspace cut by k of
    them holds k fewer (their size is found from the two sizes that M sets)."""
    sizes = [(9, 8, 7), (12, 5, 9), (6, 16, 5)]
    nb = 4
    lats, rs = [], []
    for L in sizes:
        lat, g = lattice("ti", L, (1, 0, 1))
        lats.append(lat)
        rs.append(start(lat, nb, torch.complex128, g))
    batch = pv.Batch(lats)
    pv.pv_batch_set_tuning(batch, pv.PV_C128, nb, {"kernel": kernel})
    size = lambda m: pv.lib().pv_batch_kpm_workspace_size(batch.handle, pv.PV_C128, nb, m)   # noqa: E731
    mom = lambda m: up(len(lats) * nb * m * 8)   # noqa: E731
    pb = (size(16) - mom(16)) - (size(14) - mom(14))   # 8 and 7 buffers
    full, have = size(M), min(64, M // 2)
    least = full - (have - 2) * pb
    a, b = (ctypes.c_double * 3)(9.0, 9.5, 10.0), (ctypes.c_double * 3)(0.0, 0.1, -0.1)
    ptrs = (ctypes.c_void_p * 3)(*[r.data_ptr() for r in rs])
    mus = []
    for n in sorted({full, least, least + pb, full - 1 if have > 2 else full}, reverse=True):
        for _ in range(2):   # captured, then replayed
            w = Work(n)
            mu = torch.full((3, nb, M), float("nan"), dtype=torch.float64, device="cuda")
            for _ in range(2):
                st = pv.lib().pv_batch_kpm_moments(batch.handle, pv.PV_C128, nb, M, a, b, ptrs,
                                                   ctypes.c_void_p(mu.data_ptr()), w.ptr(), n, stream())
                assert st == 0, pv.lib().pv_last_error()
                w.check()
            mus.append(mu)
    for mu in mus[1:]:
        assert (mu - mus[0]).abs().max() <= 1e-12
    w = Work(least)
    assert pv.lib().pv_batch_kpm_moments(batch.handle, pv.PV_C128, nb, M, a, b, ptrs, ctypes.c_void_p(mu.data_ptr()),
                                         w.ptr(), least - 1, stream()) == 4
