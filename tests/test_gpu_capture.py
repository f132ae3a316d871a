"""Steps, initial states and moments captured into a graph.

lbm_step, lbm_init_* and lbm_moments only launch kernels, so a program may
capture them and replay the graph among eager calls. A replay names the two
population buffers that the capture saw; the state therefore has to be in the
same one again after every even number of steps, captured or eager, before and
after the capture, whether the grid takes its steps singly or in pairs. The
reference is a handle that makes the same steps one call at a time, eagerly:
pairs and single steps have the same bits.
"""
import pytest
import torch

import paper_2112_08479_amd as pkg

GRIDS = [(128, 8, 16, 0, pkg.F32), (512, 32, 64, 0, pkg.F32), (385, 30, 64, 0, pkg.F64)]


def _pair(nx, ny, nz, model, storage):
    cfg = pkg.Config(nx, ny, nz, model=model, storage=storage, re_b=5000.0, cs_smag=0.1)
    stream = torch.cuda.Stream()
    out = pkg.Lattice(cfg, stream=stream), pkg.Lattice(cfg, stream=stream), stream
    for lat in out[:2]:
        lat.init_lock_exchange(0.25, 1e-3, 3)
    return out


def _singles(lat, n):
    for _ in range(n):
        lat.step(1)


def _capture(stream, body):
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        body()

    def replay():
        with torch.cuda.stream(stream):
            graph.replay()
        stream.synchronize()
    return replay


def _same(a, b, stream):
    with torch.cuda.stream(stream):
        x, y = a.moments(pkg.OUT_F64), b.moments(pkg.OUT_F64)
    stream.synchronize()
    return all(torch.equal(x[k], y[k]) for k in x) and bool(torch.isfinite(x["ux"]).all())


@pytest.mark.gpu
@pytest.mark.parametrize("grid", GRIDS)
@pytest.mark.parametrize("n", [2, 4, 6])
def test_replayed_steps_go_on_from_each_other_and_from_eager_ones(grid, n):
    lat, ref, stream = _pair(*grid)
    lat.step(2)  # before the capture
    _singles(ref, 2)
    replay = _capture(stream, lambda: lat.step(n))
    for eager in (0, 2, 6, 4):
        replay()
        _singles(ref, n)
        assert _same(lat, ref, stream), eager
        lat.step(eager)
        _singles(ref, eager)
        assert _same(lat, ref, stream), eager
    lat.close()
    ref.close()


@pytest.mark.gpu
@pytest.mark.parametrize("grid", GRIDS)
@pytest.mark.parametrize("warmup", [2, 3, 4, 5, 6])
def test_a_graph_of_steps_serves_a_fresh_start(grid, warmup):
    lat, ref, stream = _pair(*grid)
    lat.step(warmup)
    lat.step(warmup % 2)
    replay = _capture(stream, lambda: lat.step(2))
    for _ in range(2):
        lat.init_lock_exchange(0.25, 1e-3, 3)
        ref.init_lock_exchange(0.25, 1e-3, 3)
        for _ in range(3):
            replay()
            _singles(ref, 2)
            assert _same(lat, ref, stream)
    lat.close()
    ref.close()


@pytest.mark.gpu
@pytest.mark.parametrize("grid", GRIDS)
def test_captured_moments_and_initial_states(grid):
    lat, ref, stream = _pair(*grid)
    out = {}
    with torch.cuda.stream(stream):
        lat.moments()
    moments = _capture(stream, lambda: out.update(lat.moments(pkg.OUT_F64)))
    start = _capture(stream, lambda: (lat.init_lock_exchange(0.25, 1e-3, 3), lat.step(2)))
    for n in (2, 4, 6, 2):
        start()
        ref.init_lock_exchange(0.25, 1e-3, 3)
        _singles(ref, 2)
        lat.step(n)
        _singles(ref, n)
        moments()
        with torch.cuda.stream(stream):
            want = ref.moments(pkg.OUT_F64)
        stream.synchronize()
        assert all(torch.equal(out[k], want[k]) for k in want), n
    lat.close()
    ref.close()
