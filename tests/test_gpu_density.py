"""The FP64 charge density against the oracle's where its tiled kernel can go
wrong: particles strayed from their tiles in mid-cycle, ragged tiles, a tile
holding more particles than a pass takes, weights of very different size in
one box, and the ends of a moving window.

Tolerance: positions are exported as (cell + offset) dx, so the oracle
recovers a cell coordinate below 128 to two roundings, 128 * 2^-52 = 3e-14
cells; the weights' slope is at most one per axis, so a node differs by at
most 3 * 3e-14 of the charge of the particles that reach it, at most that of
the densest node's neighbourhood: 1e-12 of max |rho| leaves a factor of ten."""
import dataclasses

import numpy as np
import pytest

from parity import oracle_grid

pytestmark = pytest.mark.gpu

CASES = [
    # nx, order, tile, sort interval, steps
    ((37, 23), 1, (8, 8), 4, 7),        # ragged tiles, three steps into a cycle
    ((37, 23), 2, (16, 8), 3, 3),       # right after a check
    ((40, 24), 3, (8, 12), 4, 6),
    ((11, 13, 9), 1, (4, 5, 6), 1, 2),
    ((12, 9, 14), 2, (4, 9, 5), 2, 3),
    ((12, 9, 14), 3, (12, 9, 14), 1, 2),  # one tile: a region wider than the box
]


def _plasma(nx, dx, seed):
    rng = np.random.default_rng(seed)
    dim = len(nx)
    n = 4 * int(np.prod(nx))
    x = rng.random((n, dim)) * np.asarray(nx) * np.asarray(dx)
    # 2,500 particles in one cell: several passes over one tile
    xd = (np.asarray([n // 2 for n in nx]) + rng.random((2500, dim))) * np.asarray(dx)
    x = np.concatenate([x, xd])
    u = rng.normal(0, 0.4, (len(x), 3))
    w = -10.0 ** rng.uniform(-7, 0, len(x))
    return x, u, w


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c[0])) + f"_o{c[1]}")
def test_density_matches_oracle(orc, case):
    from paper_1503_00276_amd import pic

    nx, order, tile, si, steps = case
    dx = (0.2, 0.25, 0.22)[:len(nx)]
    cfg = pic.Config(ndim=len(nx), nx=nx, dx=dx, dt=0.1, shape_order=order, tile=tile, sort_interval=si,
                     ion_density=0.3)
    sim = pic.Pic(cfg)
    sim.load_particles(*_plasma(nx, dx, 3 + order), rqm=-1.0)
    sim.load_particles(*_plasma(nx, dx, 9), rqm=2.0, species=2)
    print("density", case, flush=True)
    sim.step(steps)
    x, _, w = sim.state()
    ref = orc.rho(oracle_grid(orc, cfg), x, w) + 0.3
    rho = sim.rho()
    np.testing.assert_allclose(rho, ref, rtol=0, atol=1e-12 * np.abs(ref).max())
    sim.close()


@pytest.mark.parametrize("order", [1, 2, 3])
def test_density_at_the_window_ends(orc, order):
    """Charge that reaches nodes beyond the window is dropped, on both ends,
    also where the window's seam lies inside a tile."""
    from paper_1503_00276_amd import pic

    nx, dx = (24, 16), (0.2, 0.25)
    rng = np.random.default_rng(order)
    n = 3 * nx[0] * nx[1]
    x = rng.random((n, 2)) * np.asarray(nx) * np.asarray(dx)
    cfg = pic.Config(ndim=2, nx=nx, dx=dx, dt=0.1, shape_order=order, tile=(8, 8), move_window=1,
                     inject_ppc=(2, 2, 1), inject_w=-0.25)
    sim = pic.Pic(cfg)
    sim.load_particles(x, rng.normal(0, 0.3, (n, 3)), np.full(n, -0.3), rqm=-1.0)
    sim.step(7)
    xs, _, w = sim.state()
    shifts = int(np.floor(7 * cfg.dt / dx[0]))
    # the window inside a wider periodic box, four empty columns on either side
    g = dataclasses.replace(oracle_grid(orc, cfg), nx=(nx[0] + 8, nx[1]), xmin=(0.0, 0.0, 0.0), window=0)
    xw = xs + np.asarray([(4 - shifts) * dx[0], 0.0])
    ref = orc.rho(g, xw, w).reshape(nx[1], nx[0] + 8)[:, 4:-4].reshape(-1)
    rho = sim.rho()
    # (a lab position below 64 cells, moved to the window: two more roundings)
    np.testing.assert_allclose(rho, ref, rtol=0, atol=1e-12 * np.abs(ref).max())
    sim.close()
