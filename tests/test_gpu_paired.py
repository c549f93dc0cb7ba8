"""GPU parity of the staged kernels whose elements are two neighbouring
complex64 columns: against the explicit matrix, and against the kernels with
one column per element, which the same call takes when its output is not
aligned to 16 bytes.

Tolerances: both kernels do the same operations on every number, so vectors
are equal bit for bit; the FP64 dots differ by the order of their sums
(n * 1.1e-16 of the sum of moduli, n < 1e5: 2e-11).  Against the matrix: a step
rounds at most 24 times (20 products and the epilogue) at eps = 6e-8, of the
largest entry: 1.5e-6."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1708_09689_amd as pv  # noqa: E402
import workloads as W  # noqa: E402

from gpu_common import Case, dev, host, rel_err  # noqa: E402
from test_gpu_codegen import GenCase  # noqa: E402


def halfway(t):
    """The block in storage that starts 8 bytes after a 16-byte boundary."""
    buf = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)
    out = buf[1:].view(t.shape)
    out.copy_(t)
    assert out.data_ptr() % 16 == 8
    return out


LATTICES = [("ti", (5, 4, 9), (1, 1, 0)), ("ti", (37, 3, 6), (0, 1, 1)), ("weyl", (21, 6, 5), (1, 0, 1)),
            ("graphene4", (33, 11), (0, 1)), ("graphene2", (75, 9), (1, 0)),
            ("xz", (13, 4, 6), (1, 0, 1)), ("2d", (35, 9), (0, 1))]   # generated kernels: the last two


@pytest.mark.parametrize("name,L,per", LATTICES)
@pytest.mark.parametrize("nb", [2, 4, 32])
@pytest.mark.parametrize("elems,wg", [(2, 0), (2, 512), (4, 0), (4, 512)])
def test_pairs_of_columns_equal_single_columns(name, L, per, nb, elems, wg):
    generated = name in ("xz", "2d")
    if generated and (elems, wg) not in ((2, 0), (4, 512)):
        pytest.skip("generated kernels: the smallest and the largest tile")
    c = (GenCase if generated else Case)(name, L, per, seed=41, vdtype=np.float32)
    pv.pv_lattice_set_tuning(c.lat, pv.PV_C64, nb, {"kernel": 2, "elems_per_lane": elems, "workgroup_size": wg})
    xh, zh = (W.gaussian_block(c.H.shape[0], nb, W.generator(42, i), np.complex64) for i in (1, 2))
    x, z = dev(xh), dev(zh)
    h = c.H @ xh.astype(np.complex128) - 0.25 * xh
    for gamma, flags in ((0.0, 0), (-1.0, 0), (-1.0, 7)):
        y = torch.zeros_like(x)
        w = halfway(y)
        dy = pv.pv_spmmv(c.lat, x, y, 0.5, 0.25, gamma, z=z, dot_flags=flags)
        dw = pv.pv_spmmv(c.lat, x, w, 0.5, 0.25, gamma, z=z, dot_flags=flags)
        assert rel_err(host(y), 0.5 * h + gamma * zh) < 1.5e-6
        assert np.array_equal(host(y), host(w))
        if flags:
            size = (np.abs(xh) ** 2).sum(0).max() + (np.abs(host(y)) ** 2).sum(0).max()
            assert np.abs(host(dy) - host(dw)).max() < 2e-11 * size
    coef = np.array([0.5, 0.3 - 0.1j, 0.2j, -0.1, 0.05])
    y = torch.zeros_like(x)
    w = halfway(y)
    pv.pv_cheb_series(c.lat, x, y, 9.0, 0.1, coef)
    pv.pv_cheb_series(c.lat, x, w, 9.0, 0.1, coef)
    assert np.array_equal(host(y), host(w))


@pytest.mark.parametrize("name,L,nb", [("ti", (64, 64, 64), 1), ("ti", (64, 64, 64), 2), ("weyl", (61, 67, 70), 4),
                                       ("graphene4", (300, 301), 16)])
@pytest.mark.parametrize("M", [2, 4, 6, 160])
def test_kpm_of_start_vectors_off_alignment(name, L, nb, M):
    """The steps that read a start block 8 bytes off a 16-byte boundary take
    another kernel, with another number of partial sums, than the others.  Both
    runs round every number alike up to the contraction of single operations:
    at unit norm, M steps of 24 roundings at eps = 6e-8 summed over random
    signs, sqrt(M) * 24 * eps < 2e-5."""
    c = Case(name, L, (1,) * len(L), seed=43, vdtype=np.float32)
    assert c.D * nb >= 1 << 20
    r = dev(c.block(nb, kind="phase", dtype=np.complex64))
    a = 9.0
    ref = host(pv.pv_kpm_moments(c.lat, r, M, a, 0.0))
    mu = host(pv.pv_kpm_moments(c.lat, halfway(r), M, a, 0.0))
    assert np.abs(mu - ref).max() < 2e-5
