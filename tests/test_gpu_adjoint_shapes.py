"""Gradients under launch shapes of two numbers per lane and 512 lanes (what the
autotuner picks for KPM steps) equal the direct kernel's: the adjoint steps take
the staged kernel's tile of their own whatever the shape says, and drop the
walk, strip and workgroup fields that belong to another tile.  Tolerance:
complex128, sums of at most a few hundred products in another order, 1e-12 of
the largest gradient entry."""

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1708_09689_amd as pv  # noqa: E402

from gpu_common import MODELS  # noqa: E402


@pytest.mark.parametrize("name,L,per,nb", [("ti", (70, 64, 61), (1, 0, 1), 1), ("ti", (33, 10, 9), (0, 1, 1), 4),
                                           ("weyl", (65, 66, 70), (1, 1, 0), 2), ("graphene4", (259, 255), (1, 0), 8)])
@pytest.mark.parametrize("shape", [{"kernel": 0, "elems_per_lane": 2}, {"kernel": 2, "elems_per_lane": 2},
                                   {"kernel": 2, "elems_per_lane": 2, "workgroup_size": 512, "walk_planes": 3,
                                    "strip_rows": 2, "groups_per_xcd": 16},
                                   {"kernel": 2, "elems_per_lane": 1, "walk_planes": 4, "groups_per_xcd": 8}])
def test_gradient_under_longer_tiles(name, L, per, nb, shape):
    code, params, _ = MODELS[name]
    st = pv.pv_model_stencil(code, params)
    lat = pv.Lattice(L, per, st)
    g = torch.Generator(device="cuda").manual_seed(18)
    n_field = lat.n_rows if st["pot_mode"] == pv.PV_POT_ORBITAL else lat.n_sites
    V = torch.rand(n_field, dtype=torch.float64, device="cuda", generator=g).requires_grad_()
    r = torch.randn(lat.n_rows, nb, dtype=torch.complex128, device="cuda", generator=g)
    M = 10
    gbar = torch.randn(nb, M, dtype=torch.float64, device="cuda", generator=g)
    out = []
    for t in ({"kernel": 1}, shape):
        pv.pv_lattice_set_tuning(lat, pv.PV_C128, nb, t)
        mu = pv.kpm_moments(V, lat, r, M, 9.0, 0.1, 3)
        out.append((mu.detach(), torch.autograd.grad(mu, V, gbar)[0]))
    for a, b in zip(*out):
        assert (a - b).abs().max() <= 1e-12 * a.abs().max()
