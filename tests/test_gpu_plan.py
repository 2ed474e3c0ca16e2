"""Runs whose step count the selected variant does not divide, after autotuning
(the launches are then chosen from the launch times), against one launch per
step bit for bit; batches whose instances have waves at the walls, away from
them and both."""
import numpy as np
import pytest

import synth

gpu = pytest.mark.gpu
NMAX = 23


def _torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@gpu
@pytest.mark.parametrize("bc,nx,ny", [(synth.PERIODIC, 1000, 333), (synth.DIRICHLET, 640, 500),
                                      (synth.PERIODIC, 200, 90)])
def test_planned_runs_bitwise_equal_single_steps(bc, nx, ny):
    torch = _torch()
    from paper_2408_01081_amd.lbm import Lattice
    prob = synth.plane_wave_problem(nx, ny, bc, seed=3, kmax=3)
    v0, s0 = (torch.from_numpy(a) for a in prob.initial_fields())
    W, T = (torch.from_numpy(a) for a in prob.wall_table(NMAX))
    lat = Lattice(prob.nx, prob.ny, prob.dx, prob.dt, prob.lam, prob.mu, prob.rho, prob.bc)

    def start():
        lat.init(v0, s0)
        if bc == synth.DIRICHLET:
            lat.set_wall_velocity(W, T)

    start()
    ref = []
    for _ in range(NMAX):
        ref.append(lat.step(1).populations())
    start()
    lat.autotune(reps=5, use_cache=False)
    for n in range(1, NMAX + 1):
        start()
        assert torch.equal(lat.step(n).populations(), ref[n - 1]), n


@gpu
def test_planned_batch_runs_bitwise_equal_single_steps():
    torch = _torch()
    from paper_2408_01081_amd.batch import Batch
    g = np.random.default_rng(0)
    sizes = [(64, 64), (50, 24), (114, 62), (115, 40), (200, 130), (33, 17), (300, 100), (151, 38)]
    insts = [dict(nx=nx, ny=ny, dx=0.1, dt=0.02, lam=1.0, mu=0.7, rho=1.3, bc=(i + k) % 2)
             for k in range(2) for i, (nx, ny) in enumerate(sizes)]
    b = Batch(insts)
    v = torch.from_numpy(g.standard_normal(2 * b.total_nodes)).cuda()
    s = torch.from_numpy(g.standard_normal(3 * b.total_nodes)).cuda()
    b.init(v, s)
    ref = []
    for _ in range(NMAX):
        b.step(1)
        ref.append(b.moments().clone())
    # every variant, and the launches chosen from the launch times
    for cfg in [c["index"] for c in b.tblock_configs()] + [None]:
        if cfg is None:
            b.init(v, s)
            b.autotune(reps=3)
        else:
            b.tblock_config = cfg
        for n in range(1, NMAX + 1):
            b.init(v, s)
            b.step(n)
            assert torch.equal(b.moments(), ref[n - 1]), (cfg, n)
