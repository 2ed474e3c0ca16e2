"""Runs with a body load under a selected tile variant: periodic lattices with
more tiles than pay take the sweeps with extras, fewer tiles and lattices with
walls the tiles; the steps are those of one launch per step either way."""
import numpy as np
import pytest

import synth

gpu = pytest.mark.gpu


def _torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


# (nx, ny, rank, displacement, boundary, whether tiles): 54 x 6 nodes stored by
# a tile of 5 steps with a load, so 256 tiles are 2 x 128 (108 x 768), 512 are
# 4 x 128, 1024 are 8 x 128
CASES = [(108, 768, 32, False, synth.PERIODIC, True), (108, 769, 32, False, synth.PERIODIC, False),
         (216, 768, 32, True, synth.PERIODIC, True), (217, 768, 17, True, synth.PERIODIC, False),
         (216, 769, 16, True, synth.PERIODIC, False), (432, 768, 16, False, synth.PERIODIC, True),
         (433, 768, 3, False, synth.PERIODIC, False), (108, 769, 32, False, synth.DIRICHLET, True),
         (216, 769, 32, True, synth.DIRICHLET, True), (450, 800, 0, True, synth.PERIODIC, True)]


@gpu
@pytest.mark.parametrize("nx,ny,R,disp,bc,tiles", CASES)
def test_loaded_runs_leave_tiles_where_sweeps_are_faster(nx, ny, R, disp, bc, tiles):
    torch = _torch()
    from paper_2408_01081_amd.lbm import Lattice
    g = np.random.default_rng(R)
    nmax = 13
    lat = Lattice(nx, ny, 0.1, 0.02, 1.0, 0.7, 1.3, bc, displacement=disp)
    if R:
        lat.set_body_force(*(torch.from_numpy(a) for a in (
            0.5 * g.standard_normal((R, 2, nx)), g.standard_normal((R, ny)),
            g.standard_normal((nmax + 1, R)))))
    v0 = torch.from_numpy(g.standard_normal((2, ny, nx)))
    s0 = torch.from_numpy(g.standard_normal((3, ny, nx)))
    u0 = torch.from_numpy(g.standard_normal((2, ny, nx)))

    def run(cfg, step):
        lat.init(v0, s0)
        if disp:
            lat.init_displacement(u0)
        lat.tblock_config = cfg
        for _ in range(nmax // step):
            lat.step(step)
        return [lat.populations()] + ([lat.displacement()] if disp else [])

    cfg = [c for c in lat.tblock_configs() if c["seg_rows"] == -1016 and c["steps"] == 5][0]
    ref, got = run(-1, 1), run(cfg["index"], nmax)
    for a, b in zip(got, ref):
        assert torch.equal(a, b)
    assert (lat.steps_per_launch == 5) == tiles, lat.steps_per_launch
