"""Blocked steps of small lattices (a workgroup per tile, tile in registers):
shapes just below, at and just above one tile's stored columns and rows, every
number of steps of a run, with and without a body load and the displacement
state, against one launch per step bit for bit."""
import numpy as np
import pytest

import synth

gpu = pytest.mark.gpu


def _torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@gpu
@pytest.mark.parametrize("bc", [synth.PERIODIC, synth.DIRICHLET])
@pytest.mark.parametrize("R,disp", [(0, False), (16, False), (32, False), (0, True), (17, True)])
def test_tile_edges_bitwise_equal_single_steps(bc, R, disp):
    torch = _torch()
    from paper_2408_01081_amd.lbm import Lattice
    nmax = 19
    g = np.random.default_rng(R)
    probe = Lattice(64, 64, 0.1, 0.02, 1.0, 1.0, 1.0, bc)
    tiles = [c for c in probe.tblock_configs() if c["seg_rows"] < -1000]
    assert len(tiles) == 4
    for c in tiles:
        T, cols = c["steps"], 64 - 2 * c["steps"]
        for nx, ny in [(cols, 8), (cols - 1, 7), (cols + 1, 25), (2 * cols + 1, 15)]:
            dx, dt = 0.1, 0.02
            lat = Lattice(nx, ny, dx, dt, 1.0, 0.7, 1.3, bc, displacement=disp)
            if R:
                lat.set_body_force(*(torch.from_numpy(a) for a in (
                    0.5 * g.standard_normal((R, 2, nx)), g.standard_normal((R, ny)),
                    g.standard_normal((nmax + 1, R)))))
            v0 = torch.from_numpy(g.standard_normal((2, ny, nx)))
            s0 = torch.from_numpy(g.standard_normal((3, ny, nx)))
            u0 = torch.from_numpy(g.standard_normal((2, ny, nx)))

            def run(cfg, counts):
                lat.init(v0, s0)
                if disp:
                    lat.init_displacement(u0)
                lat.tblock_config = cfg
                out = []
                for n in counts:
                    lat.step(n)
                    out.append([lat.populations()] + ([lat.displacement()] if disp else []))
                return out

            ref = run(-1, [1] * nmax)
            for n in (1, 2, T - 1, T, T + 1, 2 * T + 1, nmax):
                got = run(c["index"], [n])[-1]
                for a, b in zip(got, ref[n - 1]):
                    assert torch.isfinite(a).all()
                    assert torch.equal(a, b), (c, nx, ny, n)
