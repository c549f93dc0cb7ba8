"""GPU parity of staged sweeps whose walks the launch rule chooses: along y on
lattices of a few planes z, and in chunks that fill the last round of walks.
Against the explicit matrix (complex128 1e-13, complex64 2e-6 of the largest
entry, as for every staged sweep), and bit for bit against walks along z in the
fewest chunks, which a launch with a strip height of its own keeps; FP64 dots up
to the order of their sums (n * 1.1e-16 of the sum of moduli, n < 2e5: 2e-11)."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1708_09689_amd as pv  # noqa: E402

from gpu_common import Case, dev, host, rel_err  # noqa: E402

LATTICES = [("ti", (33, 64, 1), (1, 1, 1), 32), ("ti", (70, 64, 2), (0, 1, 1), 32), ("ti", (70, 40, 3), (1, 0, 0), 32),
            ("ti", (130, 60, 4), (1, 1, 0), 32), ("ti", (200, 41, 5), (0, 1, 1), 16), ("ti", (61, 100, 7), (1, 0, 1), 32),
            ("weyl", (64, 90, 6), (1, 1, 0), 32), ("weyl", (130, 75, 4), (0, 0, 1), 32),
            ("ti", (57, 83, 11), (1, 1, 1), 8), ("graphene4", (97, 103), (1, 0), 16)]


@pytest.mark.parametrize("name,L,per,nb", LATTICES)
@pytest.mark.parametrize("dtype", [np.complex128, np.complex64])
@pytest.mark.parametrize("longest", [False, True])
def test_chosen_walks_equal_walks_along_z(name, L, per, nb, dtype, longest):
    c128 = dtype == np.complex128
    c = Case(name, L, per, seed=51, vdtype=np.float64 if c128 else np.float32)
    code = pv.PV_C128 if c128 else pv.PV_C64
    shape = {"kernel": 2, "elems_per_lane": (1 if c128 else 2) * (2 if longest else 1),
             "workgroup_size": 512 if longest else 0}
    xh, zh = c.block(nb, dtype=dtype), c.block(nb, seed=2, dtype=dtype)
    x, z = dev(xh), dev(zh)
    coef = np.array([0.5, 0.3 - 0.1j, 0.2j, -0.1, 0.05])
    outs = []
    for own in (0, 4):
        pv.pv_lattice_set_tuning(c.lat, code, nb, dict(shape, strip_rows=own))
        y = [torch.empty_like(x) for _ in range(3)]
        pv.pv_spmmv(c.lat, x, y[0], 0.5, 0.25, 0.0)
        d = pv.pv_spmmv(c.lat, x, y[1], 0.5, 0.25, -1.0, z=z, dot_flags=7)
        pv.pv_cheb_series(c.lat, x, y[2], 9.0, 0.1, coef)
        outs.append((y, host(d)))
    ref = 0.5 * (c.H @ xh.astype(np.complex128) - 0.25 * xh)
    tol = 1e-13 if c128 else 2e-6
    assert rel_err(host(outs[0][0][0]), ref) < tol
    assert rel_err(host(outs[0][0][1]), ref - zh) < tol
    for a, b in zip(outs[0][0], outs[1][0]):
        assert torch.equal(a, b)
    assert np.abs(outs[0][1] - outs[1][1]).max() < 2e-11 * np.abs(outs[1][1]).max()
