"""Steps taken two at a time against single steps: the same bits.

lbm_step takes pairs of steps on grids large enough for it, so a run in one call
must leave the populations that the same number of calls of one step leaves.
About half of the grids below pair; the others hold single steps to themselves.
test_gpu_pairs.py has the grids that are asserted to pair and holds their single
steps to the oracle, as test_gpu_fullsize.py does; those of test_gpu_parity.py
are too small to pair.
"""
import numpy as np
import pytest

import paper_2112_08479_amd as pkg

CLOSURES = {"les": dict(cs_smag=0.1), "none": {}, "printed": dict(cs_smag=0.03, sc_t=0.03, smag_paper_form=True),
            "general": dict(cs_smag=0.1, omega3=1.2, omega4=0.9, omega5=1.1, omega6=0.8),
            "param": dict(parametrized=True, limiter=1e-2)}


@pytest.mark.gpu
@pytest.mark.parametrize("grid,model,storage,closure", [
    ((512, 32, 64), 0, pkg.F32, "les"), ((513, 33, 65), 0, pkg.F32, "none"), ((447, 31, 63), 0, pkg.F32, "param"),
    ((449, 25, 66), 0, pkg.F32, "general"), ((511, 23, 64), 1, pkg.F32, "printed"), ((513, 24, 67), 1, pkg.F32, "none"),
    ((449, 33, 63), 2, pkg.F32, "les"), ((512, 31, 64), 2, pkg.F32, "param"), ((513, 26, 65), 0, pkg.F64, "les"),
    ((447, 24, 64), 0, pkg.F64, "param"), ((449, 31, 63), 1, pkg.F64, "printed"),
])
def test_pairs_of_steps_are_single_steps(grid, model, storage, closure):
    import torch
    nx, ny, nz = grid
    rng = np.random.default_rng(nx * ny + model)
    chi = torch.from_numpy(rng.random((nz, ny, nx))).cuda()
    lat = pkg.Lattice(pkg.Config(nx, ny, nz, model=model, storage=storage, re_b=5000.0, **CLOSURES[closure]))
    got = []
    for calls in ([5], [1] * 5, [2, 3]):
        lat.init_from_field(chi)
        for n in calls:
            lat.step(n)
        assert lat.step_count == 5
        got.append(lat.get_populations())
    for f, phi in (got[0], got[2]):
        assert np.array_equal(f, got[1][0]) and np.array_equal(phi, got[1][1])
    assert np.isfinite(got[0][0]).all()
    lat.close()
