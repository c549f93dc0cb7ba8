"""Which runs on 2D lattices take passes of several steps (host only): the
workspace queries ask for four vectors, not two, where passes serve the run.
Times in the comments: microseconds on an MI355X, passes and sweeps."""

import pytest

import paper_1708_09689_amd as pv


def lattice(model, L):
    return pv.Lattice(L, (0, 1), pv.pv_model_stencil(model, [1.0]))


def vectors(lat, dtype, nb, nbytes):
    vb = (lat.n_rows * nb * (16 if dtype == pv.PV_C128 else 8) + 255) // 256 * 256
    return nbytes / vb


G2, G4 = pv.PV_MODEL_GRAPHENE2, pv.PV_MODEL_GRAPHENE4


@pytest.mark.parametrize("model,L,dtype,nb,passes", [
    (G2, (1024, 1024), pv.PV_C128, 1, True),      # 32 terms: 293, 784
    (G2, (8, 20000), pv.PV_C128, 1, True),        # 638, 808
    (G2, (8, 200000), pv.PV_C128, 1, False),      # 5637, 5660
    (G4, (512, 512), pv.PV_C128, 1, True),        # 383, 458
    (G4, (8, 20000), pv.PV_C128, 1, False),       # 1277, 858
    (G4, (8, 20000), pv.PV_C128, 4, False),       # 1449, 1032
    (G4, (8, 200000), pv.PV_C128, 2, False),
    (G4, (60, 1000), pv.PV_C128, 1, False),       # 200, 171
    (G4, (16, 512), pv.PV_C128, 4, False),        # 182, 164
    (G4, (8, 20000), pv.PV_C64, 1, True),         # 656, 747
    (G4, (100000, 8), pv.PV_C128, 4, True),       # 3712, 8707
])
def test_passes_of_a_long_series(model, L, dtype, nb, passes):
    lat = lattice(model, L)
    assert vectors(lat, dtype, nb, pv.lib().pv_cheb_series_workspace_size(lat.handle, dtype, nb)) == (4 if passes else 2)


@pytest.mark.parametrize("model,L,nb,M,passes", [
    (G2, (512, 512), 1, 64, True),      # 139, 316
    (G4, (512, 512), 1, 64, True),      # 302, 430
    (G4, (8, 20000), 4, 16, False),     # 297, 238
    (G4, (8, 200000), 1, 4, False),     # 750, 379: two steps, three computed
    (G4, (8, 200000), 1, 8, False),     # 1520, 757: four steps, six computed
    (G2, (8, 200000), 1, 4, False),     # 470, 353
])
def test_passes_of_kpm_moments(model, L, nb, M, passes):
    lat = lattice(model, L)
    need = vectors(lat, pv.PV_C128, nb, pv.lib().pv_kpm_workspace_size(lat.handle, pv.PV_C128, nb, M))
    sweeps = pv.Lattice(L, (0, 1), pv.pv_model_stencil(model, [1.0]))
    pv.pv_lattice_set_tuning(sweeps, pv.PV_C128, nb, {"kernel": 1})   # a shape of the caller's runs sweeps
    least = vectors(lat, pv.PV_C128, nb, pv.lib().pv_kpm_workspace_size(sweeps.handle, pv.PV_C128, nb, M))
    assert (need > least) if passes else (need == least)
