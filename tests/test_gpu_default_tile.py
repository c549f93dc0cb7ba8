"""The tile that a launch takes without a tuned shape (longer from 2^22
elements, 512 lanes from 2^24 on long walks) computes what the shortest tile
does, on lattices just past those sizes whose rows are no whole tiles: vectors
bit for bit, FP64 dots up to the order of their sums (n * 1.1e-16 of the sum of
moduli, n < 2e5 numbers per workgroup sum: 2e-11)."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1708_09689_amd as pv  # noqa: E402

from gpu_common import MODELS, host  # noqa: E402

LATTICES = [("ti", (83, 61, 53), 4), ("ti", (97, 91, 31), 4), ("ti", (131, 101, 40), 8), ("ti", (203, 131, 5), 8),
            ("weyl", (71, 61, 61), 8), ("graphene4", (517, 509), 4), ("graphene2", (521, 511), 8)]


@pytest.mark.parametrize("name,L,nb", LATTICES)
@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64])
def test_default_tile_equals_shortest(name, L, nb, dtype):
    code, params, _ = MODELS[name]
    lat = pv.Lattice(L, (1, 0, 1)[:len(L)], pv.pv_model_stencil(code, params))
    assert lat.n_rows * nb >= 1 << 22
    g = torch.Generator(device="cuda").manual_seed(5)
    x, z = (torch.randn(lat.n_rows, nb, dtype=dtype, device="cuda", generator=g) for _ in range(2))
    n_field = lat.n_rows if pv.pv_model_stencil(code, params)["pot_mode"] == pv.PV_POT_ORBITAL else lat.n_sites
    lat.set_potential(torch.rand(n_field, dtype=torch.float64 if dtype == torch.complex128 else torch.float32,
                                 device="cuda", generator=g))
    coef = np.array([0.5, 0.3 - 0.1j, 0.2j, -0.1, 0.05])
    c = 0 if dtype == torch.complex128 else 1
    outs = []
    for t in (None, {"kernel": 2, "elems_per_lane": 1 + c}):
        pv.pv_lattice_set_tuning(lat, c, nb, t)
        y = [torch.empty_like(x) for _ in range(4)]
        pv.pv_spmmv(lat, x, y[0], 0.5, 0.25, 0.0)
        pv.pv_spmmv(lat, x, y[1], 0.5, 0.25, -1.0, z=z)
        d = pv.pv_spmmv(lat, x, y[2], 0.5, 0.25, -1.0, z=z, dot_flags=7)
        pv.pv_cheb_series(lat, x, y[3], 9.0, 0.1, coef)
        outs.append((y, host(d)))
    for i, (a, b) in enumerate(zip(outs[0][0], outs[1][0])):
        if i == 3 and len(L) == 2 and nb <= 4:
            continue   # series of 2D lattices at these widths run several steps per pass, no tiles
        assert torch.equal(a, b)
    assert np.abs(outs[0][1] - outs[1][1]).max() < 2e-11 * np.abs(outs[1][1]).max()
