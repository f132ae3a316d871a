"""Pairs of steps on grids that are known to take them.

Every row asks the library whether its grid pairs. A run in one call leaves the
populations of single steps, bit for bit, for every collision that pairs; the
single steps of such grids, which are compiled in their own way, are held to the
oracle for the collisions that no other test takes to a pairing grid: given rates
(both scalars, both types) and the FP64 forms. Bounds of the one-step tests: 1e-13
(FP64), 2e-7 (FP32), twice that for the scalar with 27 populations.
"""
import numpy as np
import pytest
import torch

import paper_2112_08479_amd as pkg
from oracle import lbm as olbm
from tests import inputs
from tests.gpu_helpers import both

RATES = dict(omega3=1.2, omega4=0.9, omega5=1.1, omega6=0.8)
CLOSURES = {"les": dict(cs_smag=0.1), "none": {}, "printed": dict(cs_smag=0.03, sc_t=0.03, smag_paper_form=True),
            "given": RATES, "given_les": dict(cs_smag=0.1, **RATES), "param": dict(parametrized=True, limiter=1e-2)}


@pytest.mark.gpu
@pytest.mark.parametrize("grid,model,storage,closure", [
    # last x-block of one column; spans and depths off the tiles (8 rows in FP32, 5 in FP64)
    ((513, 39, 80), 0, pkg.F32, "none"), ((577, 8, 97), 0, pkg.F32, "les"), ((833, 8, 106), 0, pkg.F32, "given_les"),
    ((633, 8, 124), 0, pkg.F32, "given"), ((695, 8, 69), 0, pkg.F32, "param"),
    ((577, 8, 97), 2, pkg.F32, "les"), ((513, 31, 75), 2, pkg.F32, "none"), ((256, 32, 96), 2, pkg.F32, "given"),
    ((897, 8, 134), 2, pkg.F32, "given_les"), ((1025, 8, 59), 2, pkg.F32, "param"),
    ((577, 5, 97), 0, pkg.F64, "les"), ((695, 5, 69), 0, pkg.F64, "none"), ((257, 29, 55), 0, pkg.F64, "given_les"),
    ((122, 40, 79), 0, pkg.F64, "given"), ((513, 24, 64), 0, pkg.F64, "param"),
    ((1025, 5, 59), 1, pkg.F64, "les"), ((1059, 5, 57), 1, pkg.F64, "none"), ((1025, 5, 59), 1, pkg.F64, "printed"),
])
def test_a_run_in_pairs_is_a_run_of_single_steps(grid, model, storage, closure):
    nx, ny, nz = grid
    rng = np.random.default_rng(nx * ny + model)
    chi = torch.from_numpy(rng.random((nz, ny, nx))).cuda()
    lat = pkg.Lattice(pkg.Config(nx, ny, nz, model=model, storage=storage, re_b=5000.0, **CLOSURES[closure]))
    assert lat.steps_per_launch == 2
    got = []
    for calls in ([1] * 5, [5], [2, 3]):
        lat.init_from_field(chi)
        for n in calls:
            lat.step(n)
        assert lat.step_count == 5
        got.append(lat.get_populations())
    assert np.isfinite(got[0][0]).all()
    for f, phi in got[1:]:
        assert np.array_equal(f, got[0][0]) and np.array_equal(phi, got[0][1])
    lat.close()


@pytest.mark.gpu
@pytest.mark.timeout(300)
@pytest.mark.parametrize("grid,model,storage,closure", [
    ((633, 8, 124), 0, pkg.F32, "given_les"), ((256, 32, 96), 2, pkg.F32, "given"), ((122, 40, 79), 0, pkg.F64, "given_les"),
    ((695, 5, 69), 0, pkg.F64, "les"), ((695, 5, 69), 0, pkg.F64, "param"), ((1059, 5, 57), 1, pkg.F64, "printed"),
])
def test_single_steps_of_pairing_grids_against_the_oracle(grid, model, storage, closure):
    nx, ny, nz = grid
    cfg, P = both(storage, nx=nx, ny=ny, nz=nz, model=model, re_b=2000.0, g_prime=1e-3, **CLOSURES[closure])
    f, phi = inputs.near_rest_state(P.flow.Q, P.scal.Q, (nz, ny, nx), P.flow.w.numpy(), P.scal.w.numpy(), 5, eps=1e-2)
    lat = pkg.Lattice(cfg)
    assert lat.steps_per_launch == 2
    lat.set_populations(f, phi)
    f0, phi0 = lat.get_populations()
    lat.step(1)
    f1, phi1 = lat.get_populations()
    lat.close()
    tol = 1e-13 if storage == pkg.F64 else 2e-7
    of, ophi = (x.numpy() for x in olbm.step(torch.from_numpy(f0), torch.from_numpy(phi0), P))
    assert np.abs(f1 - of).max() < tol
    assert np.abs(phi1 - ophi).max() < tol * (2 if model == 2 else 1)


@pytest.mark.gpu
@pytest.mark.parametrize("grid,model,storage,closure", [
    ((128, 8, 16), 0, pkg.F32, "les"), ((1024, 64, 32), 1, pkg.F32, "les"), ((512, 32, 64), 0, pkg.F16, "les"),
    ((512, 32, 64), 2, pkg.F64, "les"), ((655, 27, 93), 2, pkg.F32, "given"),
])
def test_grids_of_single_steps_say_so(grid, model, storage, closure):
    lat = pkg.Lattice(pkg.Config(*grid, model=model, storage=storage, re_b=5000.0, **CLOSURES[closure]))
    assert lat.steps_per_launch == 1
    lat.close()
