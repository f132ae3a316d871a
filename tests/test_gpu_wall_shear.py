"""Wall shear on both sides of the span that one block holds (8 rows): the values
and their span mean against the exported FP64 moments. The mean adds the span's
values in order; both sides agree to the rounding of a few FP64 operations
(1e-11 relative, 1e-15 for a velocity near zero)."""
import numpy as np
import pytest
import torch

import paper_2112_08479_amd as pkg
from oracle import diag as odiag
from tests.gpu_helpers import both


@pytest.mark.gpu
@pytest.mark.parametrize("nx,ny", [(64, 1), (65, 7), (130, 8), (63, 9), (1, 8), (200, 33)])
@pytest.mark.parametrize("model,storage", [(0, pkg.F64), (1, pkg.F32), (2, pkg.F32), (2, pkg.F64), (0, pkg.BF16_F16S)])
def test_wall_shear_by_span(nx, ny, model, storage):
    cfg, P = both(storage, nx=nx, ny=ny, nz=5, model=model, re_b=1000.0, g_prime=1e-3, cs_smag=0.1)
    lat = pkg.Lattice(cfg)
    lat.init_from_field(torch.from_numpy(np.random.default_rng(nx + ny).random((5, ny, nx))).cuda())
    lat.step(3)
    m = {k: v.cpu() for k, v in lat.moments(pkg.OUT_F64).items()}
    want = odiag.wall_shear(torch.stack([m["ux"], m["uy"], m["uz"]]), P)
    got = [t.cpu() for t in lat.wall_shear(pkg.OUT_F64)]
    low = [t.cpu() for t in lat.wall_shear(pkg.OUT_F32)]
    for g, w, f in zip(got, want, low):
        assert float((g - w).abs().max()) <= max(1e-11 * float(want[0].abs().max()), 1e-15)
        assert torch.equal(f, g.to(torch.float32))
    # the mean is the ordered sum of the reported values
    s = torch.zeros(nx, dtype=torch.float64)
    for y in range(ny):
        s = s + got[0][y]
    assert torch.equal(got[1], s / ny)
    lat.close()
