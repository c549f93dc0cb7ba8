"""Which instances of a stencil's generated kernels the calls load: calls that
can share one do, so that a process which ran one of them meets the others'
kernels loaded (pv_spmmv_noalloc, which never compiles, included) and a first
call compiles no more than it needs."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1708_09689_amd as pv  # noqa: E402

from test_gpu_codegen import stencil  # noqa: E402


def fresh_lattice(seed, dtype, L=(12, 9, 7), nb=4):
    """A lattice whose pattern no other lattice of the process has: the terms of
    the TI with next-nearest hops in an order of its own."""
    st, *_ = stencil("xz")
    order = np.random.default_rng(seed).permutation(len(st["offsets"]))
    st["offsets"], st["blocks"] = np.asarray(st["offsets"])[order], np.asarray(st["blocks"])[order]
    lat = pv.Lattice(L, (1, 0, 1), st)
    assert pv.pv_lattice_get_codegen(lat)
    pv.pv_lattice_set_tuning(lat, pv.PV_C128 if dtype == torch.complex128 else pv.PV_C64, nb, {"kernel": 2})
    g = torch.Generator(device="cuda").manual_seed(seed)
    lat.set_potential(torch.rand(lat.n_sites, dtype=torch.float64 if dtype == torch.complex128 else torch.float32,
                                 device="cuda", generator=g))
    x, z = (torch.randn(lat.n_rows, nb, dtype=dtype, device="cuda", generator=g) for _ in range(2))
    return lat, x, z


@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64])
def test_moments_and_sweeps_with_dots_share_an_instance(dtype):
    lat, x, z = fresh_lattice(101 if dtype == torch.complex128 else 102, dtype)
    n0 = pv.pv_codegen_instances()
    pv.pv_kpm_moments(lat, x, 8, 9.0, 0.0)
    assert pv.pv_codegen_instances() == n0 + 1
    y, w = torch.empty_like(x), torch.empty_like(x)
    d = torch.zeros((x.shape[1], 4), dtype=torch.float64, device="cuda")
    pv.pv_spmmv_noalloc(lat, x, y, 0.5, 0.25, -1.0, z=z, dot_flags=7, dots=d)
    pv.pv_lattice_set_codegen(lat, False)
    pv.pv_spmmv(lat, x, w, 0.5, 0.25, -1.0, z=z, dot_flags=7)   # the interpreted kernel
    pv.pv_lattice_set_codegen(lat, True)
    v = torch.empty_like(x)
    e = pv.pv_spmmv(lat, x, v, 0.5, 0.25, -1.0, z=z, dot_flags=7)
    assert pv.pv_codegen_instances() == n0 + 1
    assert torch.equal(y, v) and torch.equal(d, e)   # the generated kernel ran without allocation
    assert (y - w).abs().max() < (1e-12 if dtype == torch.complex128 else 1e-5) * w.abs().max()


@pytest.mark.parametrize("nb", [2, 8])
def test_complex64_blocks_off_16_bytes_share_the_instances(nb):
    """Same operations on every number whatever the alignment: equal bits, also
    in place, with guards around the misaligned blocks."""
    lat, x, z = fresh_lattice(110 + nb, torch.complex64, nb=nb)
    n = x.numel()

    def off(t, fill=7.0):
        buf = torch.full((n + 4,), fill, dtype=t.dtype, device="cuda")
        v = buf[1:1 + n].view(t.shape)
        v.copy_(t)
        assert v.data_ptr() % 16 == 8
        return buf, v

    for gamma, flags in ((-1.0, 7), (-1.0, 0), (0.0, 0)):
        y = z.clone()
        d = pv.pv_spmmv(lat, x, y, 0.5, 0.25, gamma, z=y if gamma else None, dot_flags=flags)
        n0 = pv.pv_codegen_instances()
        buf, w = off(z)
        e = pv.pv_spmmv(lat, x, w, 0.5, 0.25, gamma, z=w if gamma else None, dot_flags=flags)
        assert pv.pv_codegen_instances() == n0
        assert torch.equal(y, w) and (not flags or torch.equal(d, e))
        assert bool((buf[:1] == 7.0).all()) and bool((buf[1 + n:] == 7.0).all())
    coef = np.array([0.5, 0.3 - 0.1j, 0.2j, -0.1, 0.05, 0.02, 0.1, -0.2, 0.03])
    y = torch.empty_like(x)
    pv.pv_cheb_series(lat, x, y, 9.0, 0.1, coef)
    n0 = pv.pv_codegen_instances()
    buf, w = off(x)
    pv.pv_cheb_series(lat, x, w, 9.0, 0.1, coef)
    assert pv.pv_codegen_instances() == n0 and torch.equal(y, w)
    assert bool((buf[:1] == 7.0).all()) and bool((buf[1 + n:] == 7.0).all())


@pytest.mark.parametrize("K,instances", [(1, 1), (2, 2), (3, 2), (4, 2), (5, 2), (12, 3)])
def test_instances_of_a_series(K, instances):
    """Plain steps, accumulating steps, and the run-time epilogue of the first and
    last accumulating ones: a long series compiles three."""
    lat, x, _ = fresh_lattice(120 + K, torch.complex128)
    y, w = torch.empty_like(x), torch.empty_like(x)
    coef = np.random.default_rng(K).standard_normal(K + 1)
    n0 = pv.pv_codegen_instances()
    pv.pv_cheb_series(lat, x, y, 9.0, 0.1, coef)
    assert pv.pv_codegen_instances() == n0 + instances
    pv.pv_lattice_set_tuning(lat, pv.PV_C128, x.shape[1], {"kernel": 1})
    pv.pv_lattice_set_codegen(lat, False)
    pv.pv_cheb_series(lat, x, w, 9.0, 0.1, coef)
    assert (y - w).abs().max() < 1e-12 * w.abs().max()
