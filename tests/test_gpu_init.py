"""Initialisation at the edges of its 64 x 4 tiles, on axes of one to three
nodes (where the difference formulas change), and for batches whose blocks of
256 nodes hold several instances."""
import numpy as np
import pytest

import oracle
import synth

gpu = pytest.mark.gpu

SHAPES = [(1, 1), (1, 5), (2, 2), (3, 2), (2, 3), (3, 3), (64, 4), (65, 5), (63, 3), (129, 1),
          (16, 16)]


def _torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _fields(nx, ny, seed):
    g = np.random.default_rng(seed)
    return g.standard_normal((2, ny, nx)), g.standard_normal((3, ny, nx))


@gpu
@pytest.mark.parametrize("bc", [synth.PERIODIC, synth.DIRICHLET])
def test_init_tile_edges_match_oracle(bc):
    torch = _torch()
    from paper_2408_01081_amd.lbm import Lattice
    for i, (nx, ny) in enumerate(SHAPES):
        v0, s0 = _fields(nx, ny, i)
        args = (nx, ny, 0.1, 0.02, 1.0, 0.7, 1.3, bc)
        lat = Lattice(*args)
        lat.init(torch.from_numpy(v0), torch.from_numpy(s0))
        got = lat.populations().double().cpu().numpy()
        want = oracle.Simulation(oracle.Setup(*args), v0, s0).f
        # stored f* is rounded once (2^-24); reading f back collides it in
        # FP32: under 8 further roundings of values within 4 max|f|
        assert np.abs(got - want).max() <= 32 * 2.0 ** -24 * np.abs(want).max(), (nx, ny)


@gpu
def test_batch_init_of_small_instances_matches_single():
    torch = _torch()
    from paper_2408_01081_amd.batch import Batch
    from paper_2408_01081_amd.lbm import Lattice
    insts = [dict(nx=nx, ny=ny, dx=0.1, dt=0.02, lam=1.0, mu=0.5 + 0.1 * i, rho=1.0, bc=i % 2)
             for i, (nx, ny) in enumerate(SHAPES + SHAPES[::-1])]
    fields = [_fields(p["nx"], p["ny"], i) for i, p in enumerate(insts)]
    b = Batch(insts)
    b.init(b.pack([f[0] for f in fields]), b.pack([f[1] for f in fields]))
    got = b.unpack(b.moments(system=True), 5)
    for p, (v0, s0), u in zip(insts, fields, got):
        lat = Lattice(**p)
        lat.init(torch.from_numpy(v0), torch.from_numpy(s0))
        assert torch.equal(lat.moments_U(), u), p
