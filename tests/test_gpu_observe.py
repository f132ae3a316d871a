"""The step's cached-store form and ragged blocks, and the reporting kernels, at
the sizes where their rules change.

* one step from a random state against the oracle on grids whose buffers lie
  between the store rule's bounds (23 to 128 MB; 120 in 16-bit storage) and whose
  rows take an odd number of waves; the bounds are those of the one-step tests:
  2e-7 (FP32), 1e-13 (FP64), half a unit of the stored deviation (FP16);
* diagnostics, initial diagnostics and wall shear against the same sums taken
  from the exported FP64 moments: all sides add at most a few 1e5 FP64 terms of
  one size, so they agree to 1e-11 relative, or to the 1e-15 by which a velocity
  near zero (27 terms of the weights' size that cancel) rounds.
"""
import numpy as np
import pytest
import torch

import paper_2112_08479_amd as pkg
from oracle import diag as odiag
from oracle import lbm as olbm

from tests import inputs
from tests.gpu_helpers import both, ulp


@pytest.mark.gpu
@pytest.mark.parametrize("shape,model,storage", [
    ((40, 20, 321), 0, pkg.F32), ((31, 16, 193), 0, pkg.F64), ((40, 21, 257), 1, pkg.F32), ((60, 33, 321), 0, pkg.F16),
])
def test_one_step_with_cached_stores(shape, model, storage):
    nz, ny, nx = shape
    cfg, P = both(storage, nx=nx, ny=ny, nz=nz, model=model, re_b=2000.0, g_prime=1e-3, cs_smag=0.1)
    f, phi = inputs.near_rest_state(P.flow.Q, P.scal.Q, shape, P.flow.w.numpy(), P.scal.w.numpy(), 5, eps=1e-2)
    lat = pkg.Lattice(cfg)
    assert (23 << 20) < lat.state_bytes() < ((120 if storage == pkg.F16 else 128) << 20)
    lat.set_populations(f, phi)
    f0, phi0 = lat.get_populations()
    lat.step(1)
    f1, phi1 = lat.get_populations()
    lat.close()
    of, ophi = (x.numpy() for x in olbm.step(torch.from_numpy(f0), torch.from_numpy(phi0), P))
    tol = {pkg.F64: 1e-13, pkg.F32: 2e-7, pkg.F16: 2e-7}[storage]
    half = (0.5 if storage == pkg.F16 else 0.0)
    w = P.flow.w.numpy().reshape(-1, 1, 1, 1)
    assert (np.abs(f1 - of) <= tol + half * ulp(of - w, 10)).all()
    assert (np.abs(phi1 - ophi) <= tol + half * ulp(ophi, 10)).all()


@pytest.mark.gpu
@pytest.mark.parametrize("grid,model,storage", [
    ((513, 5, 33), 0, pkg.F32), ((256, 3, 64), 1, pkg.F64), ((65, 9, 15), 2, pkg.F32), ((1030, 2, 16), 0, pkg.F16),
    ((70, 1, 300), 2, pkg.BF16_F16S),
])
def test_reports_are_the_sums_of_the_exported_moments(grid, model, storage):
    nx, ny, nz = grid
    cfg, P = both(storage, nx=nx, ny=ny, nz=nz, model=model, re_b=1000.0, g_prime=1e-3, cs_smag=0.1)
    lat = pkg.Lattice(cfg)
    rng = np.random.default_rng(nx + nz)
    chi0 = np.where(np.arange(nx) < nx // 8, 1.0, 0.0) * rng.uniform(0.5, 1.0, (nz, ny, nx))
    lat.init_from_field(torch.from_numpy(chi0).cuda())

    def near(a, b, scale=0.0, floor=0.0):
        assert abs(a - b) <= max(1e-11 * max(abs(b), scale), floor), (a, b)

    for steps in (0, 7):
        lat.step(steps)
        m = {k: v.cpu() for k, v in lat.moments(pkg.OUT_F64).items()}
        d = lat.diagnostics()
        u = torch.stack([m["ux"], m["uy"], m["uz"]])
        x, _ = odiag.front_position(m["chi"])
        near(d["mass"], float(m["rho"].sum()))
        near(d["chi_mass"], float(m["chi"].sum()))
        near(d["x_front"], float(x))
        near(d["umax"], float(torch.sqrt((u * u).sum(0)).max()), floor=1e-15)
        near(d["fw"], float(odiag.wall_friction(u, P)), P.nu0 * 3 * d["umax"] * nx * ny, floor=1e-15 * nx * ny)
        if steps == 0:
            near(d["mass0"], d["mass"])
            near(d["chi_mass0"], d["chi_mass"])
        tau, bar = (t.cpu() for t in lat.wall_shear(pkg.OUT_F64))
        otau, obar = odiag.wall_shear(u, P)
        for got, want in ((tau, otau), (bar, obar)):
            assert float((got - want).abs().max()) <= max(1e-11 * float(otau.abs().max()), 1e-15)
    lat.close()
