"""The fixed point of a work item's current tile (two-phase kernels) where its
bounds could fail: plasmas that move as one through tiles of more than 64 cells,
whose sums alone would set too coarse a unit, and particles whose momentum is
not a number in FP32."""
import numpy as np
import pytest

from parity import J_TOL, oracle_grid, rel_max

pytestmark = pytest.mark.gpu


def _current_error(orc, nx, order, x, u, w, dx=0.2, **kw):
    """RMS and largest error of the current of one step, relative to max |J|."""
    from paper_1503_00276_amd import pic

    cfg = pic.Config(ndim=len(nx), nx=nx, dx=(dx,) * len(nx), dt=dx / 2, shape_order=order, ion_density=1.0, **kw)
    sim = pic.Pic(cfg)
    sim.load_particles(x, u, w, rqm=-1.0)
    x0, u0, w0 = sim.state()
    E, B = sim.fields()
    ref = orc.step(oracle_grid(orc, cfg), x0, u0, w0, -1.0, E, B)
    sim.step(1)
    J, tile = sim.current(), list(sim.info().tile)
    sim.close()
    top = np.abs(ref.J).max()
    return np.sqrt(np.mean((J - ref.J) ** 2)) / top, np.abs(J - ref.J).max() / top, tile


# The reach of a node in a uniform plasma of a particle per cell is 48 particles
# (linear) or 45 (quadratic, times its peaks) whatever the tile, with 2.5
# standard deviations of a random one below 64; the sum over a 4x4x4 tile is 64
# or 36.  So the unit is that of the 4x4x4 tile or, with the quadratic shape, at
# most twice it, and the error with it (1.3: what the random counts do to it).
@pytest.mark.parametrize("order,factor", [(1, 1.3), (2, 2.0)])
@pytest.mark.parametrize("ppc", [1, 2, 4])
def test_a_drifting_plasma_keeps_its_unit_in_large_tiles(orc, order, factor, ppc):
    nx = (48, 32, 40)
    rng = np.random.default_rng(ppc)
    c = np.indices(nx).reshape(3, -1).T.repeat(ppc, 0)
    x = (c + rng.random(c.shape)) * 0.2
    u, w = np.tile((10.0, 4.0, 2.0), (len(x), 1)), np.full(len(x), -1.0 / ppc)
    print("drift", order, ppc, flush=True)
    rms, top, tile = _current_error(orc, nx, order, x, u, w)
    small, _, _ = _current_error(orc, nx, order, x, u, w, tile=(4, 4, 4))
    print(tile, "rms %.3e, in 4x4x4 tiles %.3e" % (rms, small), flush=True)
    assert int(np.prod(tile)) > 64 and top <= J_TOL
    assert rms <= factor * small


# Tiles whose nodes are reached by all there is: the sums must not overflow.
# (Every particle in one cell, at one corner of the tile or outside it, moving
# as one along each axis or diagonally, or against each other.)
@pytest.mark.parametrize("order", [1, 2, 3])
@pytest.mark.parametrize("tile", [(8, 8, 4), (8, 4, 4), (4, 8, 8), (16, 4, 4), (4, 4, 12), (4, 16, 4)])
def test_a_dense_spot_does_not_overflow_its_node(orc, order, tile):
    nx = (16, 16, 24) if tile[2] == 12 else (16, 16, 16)
    rng = np.random.default_rng(order)
    for cell, move in [((0, 0, 0), (10, 0, 0)), ((7, 3, 3), (0, 10, 0)), ((8, 4, 4), (0, 0, -10)),
                       ((15, 15, 1), (10, 10, 10)), ((3, 7, 2), (-10, 10, -10))]:
        n = 700
        x = (np.asarray(cell) + rng.random((n, 3))) * 0.2
        u = np.tile(np.asarray(move, float), (n, 1))
        u[n // 2:] *= rng.choice([1.0, -1.0])
        rms, top, _ = _current_error(orc, nx, order, x, u, np.full(n, -0.5), tile=tile)
        assert top <= J_TOL, (tile, cell, move, top)


@pytest.mark.parametrize("nx", [(48, 40), (16, 12, 16), (32, 16, 16)], ids=lambda n: "x".join(map(str, n)))
@pytest.mark.parametrize("order", [1, 2, 3])
def test_an_infinite_momentum_does_not_take_its_neighbours_current(nx, order):
    """1e39 is finite in FP64 and infinite in FP32: the particle adds nothing to
    the current, and the others' current stays what it is without it."""
    from paper_1503_00276_amd import pic

    rng = np.random.default_rng(order)
    ppc = 2
    n = ppc * int(np.prod(nx))
    x = rng.random((n, len(nx))) * np.asarray(nx) * 0.2
    u, w = rng.normal(0, 0.3, (n, 3)), np.full(n, -1.0 / ppc)
    got = []
    for extra in (0, 1):
        sim = pic.Pic(pic.Config(ndim=len(nx), nx=nx, dx=(0.2,) * len(nx), dt=0.08, shape_order=order))
        ux = np.concatenate([u, np.full((extra, 3), [[1e39, 0.0, 1.0]])])
        print("infinite", nx, order, extra, flush=True)
        sim.load_particles(np.concatenate([x, x[:extra]]), ux, np.concatenate([w, w[:extra]]), rqm=-1.0)
        sim.step(1)
        got.append(sim.current())
        sim.close()
    assert rel_max(got[1], got[0]) <= J_TOL


# As above in tiles whose columns are not 64 classes, or that are longest along
# x3: a node's reach is 48 particles of a uniform plasma (45), times the shortest
# extent over four.
@pytest.mark.parametrize("order,factor", [(1, 1.3), (2, 2.0)])
@pytest.mark.parametrize("tile", [(12, 8, 4), (6, 8, 4), (9, 8, 4), (4, 8, 8), (4, 8, 12), (8, 4, 12), (24, 8, 4)],
                         ids=lambda t: "x".join(map(str, t)))
def test_a_drifting_plasma_keeps_its_unit_in_any_large_tile(orc, order, factor, tile):
    nx, ppc = (48, 24, 24), 1
    rng = np.random.default_rng(ppc)
    c = np.indices(nx).reshape(3, -1).T
    x = (c + rng.random(c.shape)) * 0.2
    u, w = np.tile((10.0, 4.0, 2.0), (len(x), 1)), np.full(len(x), -1.0 / ppc)
    print("drift", order, tile, flush=True)
    rms, top, _ = _current_error(orc, nx, order, x, u, w, tile=tile)
    small, _, _ = _current_error(orc, nx, order, x, u, w, tile=(4, 4, 4))
    print("rms %.3e, in 4x4x4 tiles %.3e" % (rms, small), flush=True)
    assert top <= J_TOL
    assert rms <= factor * small


@pytest.mark.parametrize("order", [1, 2])
@pytest.mark.parametrize("tile", [(12, 6, 4), (4, 6, 12), (6, 8, 8), (12, 4, 6), (6, 6, 6)],
                         ids=lambda t: "x".join(map(str, t)))
def test_a_dense_spot_does_not_overflow_its_node_in_any_tile(orc, order, tile):
    test_a_dense_spot_does_not_overflow_its_node(orc, order, tile)


# The cubic shape and the 4x4xN tiles, which take the sum alone, and odd boxes: the
# sum of a uniform plasma over a default tile is that of 64 cells at most where
# the axes have such tiles.
@pytest.mark.parametrize("nx,order", [((36, 42, 36), 3), ((12, 21, 36), 3), ((16, 12, 48), 3), ((4, 4, 48), 1),
                                      ((4, 4, 48), 2), ((16, 4, 48), 2)])
def test_default_tiles_that_take_the_sum_are_small(nx, order):
    from paper_1503_00276_amd import pic

    sim = pic.Pic(pic.Config(ndim=3, nx=nx, dx=(0.2,) * 3, dt=0.1, shape_order=order))
    rng = np.random.default_rng(1)
    n = int(np.prod(nx))
    sim.load_particles(rng.random((n, 3)) * np.asarray(nx) * 0.2, rng.normal(0, 0.1, (n, 3)), np.full(n, -1.0))
    t = sim.info().tile
    sim.close()
    peak = (1.0, 0.75, 2.0 / 3.0)[order - 1]
    sums = (order == 3) or (t[0] == 4 and t[1] == 4)
    assert not sums or t[0] * t[1] * t[2] * peak**2 <= 64.0, list(t)
