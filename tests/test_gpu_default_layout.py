"""Step parity in the layout the library picks by itself (tile, sort interval,
chunk) for boxes whose extents leave it little choice: primes, extents below
the halo, long and thin boxes, every shape order, few and many particles per
cell, windows and r-z walls; and a store that grows after its first load."""
import numpy as np
import pytest

from parity import F_TOL, J_TOL, MOM_TOL, POS_TOL, step_parity

pytestmark = pytest.mark.gpu

CASES = [
    # nx, order, ppc, extra
    ((37, 53), 2, 4, {}),
    ((5, 4), 1, 6, {}),
    ((131, 3), 3, 3, {}),
    ((66, 67), 1, 12, {"deposit": 1}),
    ((67, 34), 3, 5, {"accumulator": 2}),
    ((11, 13, 7), 1, 5, {}),
    ((17, 5, 23), 2, 1, {}),
    ((13, 19, 4), 3, 2, {}),
    ((11, 10, 9), 2, 9, {"accumulator": 2}),
    ((13, 11, 10), 1, 3, {"deposit": 1}),
]


def _plasma(nx, dx, ppc, seed):
    rng = np.random.default_rng(seed)
    n = ppc * int(np.prod(nx))
    x = rng.random((n, len(nx))) * np.asarray(nx) * np.asarray(dx)
    return x, rng.normal(0, 0.3, (n, 3)), np.full(n, -1.0 / ppc)


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c[0])) + f"_o{c[1]}_ppc{c[2]}")
def test_default_layout_parity(orc, case):
    from paper_1503_00276_amd import pic

    nx, order, ppc, extra = case
    dx = (0.2, 0.21, 0.22)[:len(nx)]
    cfg = pic.Config(ndim=len(nx), nx=nx, dx=dx, dt=0.1, shape_order=order, ion_density=1.0, **extra)
    sim = pic.Pic(cfg)
    sim.load_particles(*_plasma(nx, dx, ppc, 17), rqm=-1.0)
    i = sim.info()
    print(case, "tile", list(i.tile), "interval", i.sort_interval, "chunk", i.chunk, flush=True)
    for k in range(10):  # across a whole cycle: the halo grows with the steps since the check
        err = step_parity(orc, sim, cfg)
        assert err["pos"] <= POS_TOL and err["mom"] <= MOM_TOL, (k, err)
        assert err["J"] <= J_TOL and err["E"] <= F_TOL and err["B"] <= F_TOL, (k, err)
    # the store grows sixfold: the tile stays, the chunk follows the particles
    sim.load_particles(*_plasma(nx, dx, 5 * ppc, 18), rqm=-1.0)
    assert list(sim.info().tile) == list(i.tile)
    err = step_parity(orc, sim, cfg)
    assert err["pos"] <= POS_TOL and err["mom"] <= MOM_TOL and err["J"] <= J_TOL, err
    sim.close()


def test_an_asked_tile_keeps_the_short_interval():
    """A tile that holds what strays in the short default interval, but not in
    the long one, is taken, alone and in a batch with boxes without one."""
    from paper_1503_00276_amd import pic

    a = pic.Config(ndim=2, nx=(20, 12), dx=(0.2, 0.2), dt=0.08, shape_order=1, tile=(4, 4))
    b = pic.Config(ndim=2, nx=(40, 40), dx=(0.2, 0.2), dt=0.08, shape_order=1)
    sim = pic.Pic(a)
    assert list(sim.info().tile)[:2] == [4, 4]
    batch = pic.PicBatch([a, b])
    assert batch.info(0).sort_interval == sim.info().sort_interval
    batch.close()
    sim.close()
