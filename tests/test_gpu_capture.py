"""Runs recorded into a graph: a captured run keeps the launches that its step count
alone determines, an uncaptured one may divide its last launches by the
autotuner's times; replays after the first, with eager work between, give the
bits of single steps."""
import pytest

import synth

gpu = pytest.mark.gpu


def _torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@gpu
@pytest.mark.parametrize("nx,ny,n", [(1000, 333, 22), (200, 90, 13)])
def test_captured_runs_after_autotuning(nx, ny, n):
    torch = _torch()
    from paper_2408_01081_amd.lbm import Lattice
    prob = synth.plane_wave_problem(nx, ny, synth.PERIODIC, seed=3, kmax=3)
    v0, s0 = (torch.from_numpy(a).cuda() for a in prob.initial_fields())
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        lat = Lattice(prob.nx, prob.ny, prob.dx, prob.dt, prob.lam, prob.mu, prob.rho, prob.bc)
        lat.init(v0, s0)
        for _ in range(n):
            lat.step(1)
        want = lat.moments()
        lat.init(v0, s0)
        lat.autotune(reps=5, use_cache=False)
        lat.init(v0, s0).step(n)
        assert torch.equal(lat.moments(), want)
        out = torch.empty_like(want)
        stream.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            lat.init(v0, s0)
            lat.step(n)
            lat.moments(out)
        for _ in range(3):
            out.zero_()
            g.replay()
            assert torch.equal(out, want)
            lat.init(v0, s0).step(n)   # eager work between the replays
            assert torch.equal(lat.moments(), want)
