"""The FP64 charge density of a tile that holds heavy and light particles: a node
that only light ones reach is as accurate, for its own charge, as any other.

Tolerance: the exported position (cell + offset) dx gives the oracle a cell
coordinate below 64 to 64 * 2^-52 * 2 = 3e-14 cells; the weights' slope is at most
one per axis, so a node is off by at most 3 * 3e-14 of the charge |w| of the
particles within two cells of it: 1e-12 of that leaves a factor of ten."""
import numpy as np
import pytest

from parity import oracle_grid

pytestmark = pytest.mark.gpu


def _reach(nx, x, w, dx):
    """|w| of the particles within two cells of each node, [z, y, x] order."""
    c = tuple(np.floor(x[:, d] / dx[d]).astype(int) % nx[d] for d in range(len(nx)))
    q = np.zeros(nx[::-1])
    np.add.at(q, c[::-1], np.abs(w))
    for ax in range(q.ndim):
        q = sum(np.roll(q, k, ax) for k in range(-2, 4))
    return q.reshape(-1)


@pytest.mark.parametrize("order", [1, 2, 3])
@pytest.mark.parametrize("nx", [(24, 20), (16, 12, 14)], ids=lambda n: "x".join(map(str, n)))
@pytest.mark.parametrize("light", [1e-6, 1e-18])
def test_light_particles_beside_heavy_ones(orc, nx, order, light):
    from paper_1503_00276_amd import pic

    dim = len(nx)
    dx = (0.2, 0.25, 0.22)[:dim]
    tile = nx if dim == 2 else (16, 12, 7)
    cfg = pic.Config(ndim=dim, nx=nx, dx=dx, dt=0.1, shape_order=order, tile=tile, sort_interval=1)
    rng = np.random.default_rng(order)
    n = 600
    cell = rng.random((n, dim)) * np.asarray(nx)
    w = np.where(np.arange(n) % 2 == 0, -1.0, -light)
    cell[::2, 0] = 3.0 * rng.random(n // 2)          # heavy: columns 0 to 2
    cell[1::2, 0] = 7.0 + 3.0 * rng.random(n // 2)   # light: columns 7 to 9
    sim = pic.Pic(cfg)
    sim.load_particles(cell * np.asarray(dx), np.zeros((n, 3)), w, rqm=-1.0)
    x, _, ws = sim.state()
    ref = orc.rho(oracle_grid(orc, cfg), x, ws)
    print("light", nx, order, light, flush=True)
    err, tol = np.abs(sim.rho() - ref), 1e-12 * _reach(nx, x, ws, dx)
    assert np.count_nonzero((np.abs(ref) > 0) & (np.abs(ref) < 1e3 * light)) > 20
    assert np.all(err <= tol), (err / np.maximum(tol, 1e-300)).max()
    sim.close()
