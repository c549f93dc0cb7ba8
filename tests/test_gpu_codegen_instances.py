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
