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


@pytest.mark.parametrize("name,sizes,nb", [("ti", [(8, 8, 8)] * 3, 1), ("ti", [(24, 24, 24)] * 8, 4),
                                           ("ti", [(31, 33, 29), (16, 7, 40), (40, 32, 12)] * 4, 16),
                                           ("weyl", [(32, 32, 32), (33, 31, 30)] * 8, 16),
                                           ("graphene4", [(64, 256), (61, 250)] * 3, 16)])
@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64])
def test_default_batch_equals_single_lattices(name, sizes, nb, dtype):
    """Batches on either side of the rules that choose the staged kernel and
    its longer tile, against each lattice's direct kernel.  Moments at unit
    norm: complex128 1e-12; complex64 M steps of 24 roundings at eps = 6e-8
    summed over random signs, sqrt(M) * 24 * eps < 1e-5 for M = 12."""
    code, params, _ = MODELS[name]
    st = pv.pv_model_stencil(code, params)
    c, M = 0 if dtype == torch.complex128 else 1, 12
    g = torch.Generator(device="cuda").manual_seed(6)
    lats, rs = [], []
    for L in sizes:
        lat = pv.Lattice(L, (1, 0, 1)[:len(L)], st)
        n_field = lat.n_rows if st["pot_mode"] == pv.PV_POT_ORBITAL else lat.n_sites
        lat.set_potential(torch.rand(n_field, dtype=torch.float32 if c else torch.float64, device="cuda", generator=g))
        pv.pv_lattice_set_tuning(lat, c, nb, {"kernel": 1})
        r = torch.randn(lat.n_rows, nb, dtype=torch.complex128, device="cuda", generator=g)
        rs.append((r / torch.linalg.vector_norm(r, dim=0) * lat.n_rows ** 0.5).to(dtype))
        lats.append(lat)
    ref = [host(pv.pv_kpm_moments(lat, r, M, 9.0, 0.0)) for lat, r in zip(lats, rs)]
    for lat in lats:
        pv.pv_lattice_set_tuning(lat, c, nb, None)
    mu = host(pv.pv_batch_kpm_moments(pv.Batch(lats), rs, M, [9.0] * len(lats), 0.0))
    for i in range(len(lats)):
        assert np.abs(mu[i] - ref[i]).max() < (1e-5 if c else 1e-12)
