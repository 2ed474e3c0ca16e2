"""The passes over a lattice's nodes that read no neighbours (populations in and
out, moments, displacement) on narrow, low and ragged lattices around the 256
nodes of a workgroup, with a body load whose value differs at every node,
against the same sums in FP64."""
import numpy as np
import pytest

import synth

gpu = pytest.mark.gpu

SHAPES = [(1, 1), (1, 700), (2, 513), (5, 103), (17, 61), (255, 1), (256, 1), (257, 3), (700, 1),
          (513, 2), (300, 5), (63, 130), (65, 9),
          # states beyond 128 MiB, whose nodes are taken in grid order
          (3, 30001), (130, 9000)]


def _torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@gpu
@pytest.mark.parametrize("nx,ny", SHAPES)
def test_passes_without_neighbours(nx, ny):
    torch = _torch()
    from paper_2408_01081_amd.lbm import Lattice
    g = np.random.default_rng(nx + 1000 * ny)
    dt, rho, R = 0.02, 1.3, 3
    lat = Lattice(nx, ny, 0.1, dt, 1.0, 0.7, rho, synth.PERIODIC, displacement=True)
    X, Y, T = g.standard_normal((R, 2, nx)), g.standard_normal((R, ny)), g.standard_normal((2, R))
    lat.set_body_force(*(torch.from_numpy(a) for a in (X, Y, T)))
    f = g.standard_normal((4, 5, ny, nx)).astype(np.float32)
    u0 = g.standard_normal((2, ny, nx))
    lat.set_populations(torch.from_numpy(f))
    lat.init_displacement(torch.from_numpy(u0))
    back = lat.populations().double().cpu().numpy()
    U = lat.moments_U().double().cpu().numpy()
    fields = lat.moments().double().cpu().numpy()
    u = lat.displacement().double().cpu().numpy()
    want = f.astype(np.float64).sum(0)
    want[:2] += 0.5 * dt / rho * np.einsum("rcx,ry,r->cyx", X, Y, T[0])
    # stored f* has up to 8 roundings of values within 8 max|f|; U adds four of
    # them, and f collides them once more (16 roundings)
    tol = 512 * 2.0 ** -24 * np.abs(f).max()
    assert np.abs(back - f).max() <= tol
    assert np.abs(U - want).max() <= tol
    assert np.abs(fields[:2] - want[:2]).max() <= tol
    cK, cmu = np.sqrt(1.7 / rho), np.sqrt(0.7 / rho)
    sxx = -rho * (cK * want[2] + cmu * want[3])
    syy = -rho * (cK * want[2] - cmu * want[3])
    assert np.abs(fields[2] - sxx).max() <= 4 * tol
    assert np.abs(fields[3] - syy).max() <= 4 * tol
    assert np.abs(fields[4] + rho * cmu * want[4]).max() <= 4 * tol
    # u(t_0) = u0: the half step of velocity goes in and out again
    assert np.abs(u - u0).max() <= 2.0 ** -23 * np.abs(u0).max() + dt * tol


# rows that fill no cache line (consecutive nodes) and the first that do (tiles),
# more nodes than a workgroup's 256
@gpu
@pytest.mark.parametrize("bc", [synth.PERIODIC, synth.DIRICHLET])
@pytest.mark.parametrize("nx,ny", [(1, 300), (2, 257), (3, 171), (5, 203), (16, 33), (31, 40),
                                   (32, 40), (33, 40)])
def test_init_of_narrow_lattices(nx, ny, bc):
    torch = _torch()
    import oracle
    from paper_2408_01081_amd.lbm import Lattice
    g = np.random.default_rng(nx + 1000 * ny)
    lam, mu, rho = 1.0, 0.7, 1.3
    args = (nx, ny, 0.1, 0.02, lam, mu, rho, bc)
    v0, du = g.standard_normal((2, ny, nx)), g.standard_normal((4, ny, nx))
    tr = lam * (du[0] + du[3])
    s0 = np.stack([tr + 2 * mu * du[0], tr + 2 * mu * du[3], mu * (du[1] + du[2])])
    lat = Lattice(*args)
    lat.init(torch.from_numpy(v0), torch.from_numpy(s0))
    got = lat.populations().double().cpu().numpy()
    want = oracle.Simulation(oracle.Setup(*args), v0, s0).f
    # as in tests/test_gpu_init.py: one rounding stored, under 8 when read
    tol = 32 * 2.0 ** -24 * np.abs(want).max()
    assert np.abs(got - want).max() <= tol
    # from the displacement gradient: the same U0, formed in FP64
    lat.init_from_gradient(torch.from_numpy(v0), torch.from_numpy(du))
    assert np.abs(lat.populations().double().cpu().numpy() - want).max() <= tol
