"""GPU parity of the periodic 3D field step at the sizes where its kernel
changes (16x4x4 tiles, or runs of 8, 16 and 32 planes marching along z), on
extents that leave ragged tiles, columns and runs, against the oracle's FP64
solve; and a batch that holds boxes of both kinds."""
import numpy as np
import pytest

from parity import F_TOL, oracle_grid

pytestmark = pytest.mark.gpu

SIZES = [
    (5, 3, 2),        # smaller than a tile: tiles
    (47, 21, 19),     # ragged tiles
    (130, 65, 53),    # 45 columns of 7 runs of 8 planes: under 512, tiles
    (130, 65, 97),    # 13 runs: 585 workgroups, runs of 8 planes
    (250, 129, 66),   # 136 columns, 9 runs: 8 planes
    (257, 130, 121),  # 153 columns, 8 runs of 16 planes, the last one short
    (257, 250, 130),  # 288 columns, 5 runs of 32 planes, the last one short
]


def _check(orc, sim, cfg, inst=()):
    g = oracle_grid(orc, cfg)
    E, B = sim.fields(*inst)
    sim.step(1)
    Eg, Bg = sim.fields(*inst)
    Bh = orc.yee_b(g, E, B, 0.5 * cfg.dt)
    En = orc.yee_e(g, E, Bh, np.zeros((3, cfg.ncell)), cfg.dt)
    Bn = orc.yee_b(g, En, Bh, 0.5 * cfg.dt)
    assert np.abs(Eg - En).max() <= F_TOL * np.abs(En).max()
    assert np.abs(Bg - Bn).max() <= F_TOL * np.abs(Bn).max()


def _cfg(pic, nx):
    return pic.Config(ndim=3, nx=nx, dx=(0.05, 0.06, 0.07), dt=0.02, shape_order=1)


def _fields(cfg, seed):
    rng = np.random.default_rng(seed)
    return rng.normal(0, 1, (3, cfg.ncell)), rng.normal(0, 1, (3, cfg.ncell))


@pytest.mark.parametrize("nx", SIZES, ids=lambda n: "x".join(map(str, n)))
def test_field_step_at_the_dispatch_edges(orc, nx):
    from paper_1503_00276_amd import pic

    print("field step", nx, flush=True)
    cfg = _cfg(pic, nx)
    sim = pic.Pic(cfg)
    sim.load_fields(*_fields(cfg, 5))
    for _ in range(2):
        _check(orc, sim, cfg)
    sim.close()


def test_batch_of_boxes_of_both_kinds(orc):
    from paper_1503_00276_amd import pic

    cfgs = [_cfg(pic, nx) for nx in [(47, 21, 19), (130, 65, 97), (20, 20, 20)]]
    sim = pic.PicBatch(cfgs)
    for k, c in enumerate(cfgs):
        sim.load_fields(k, *_fields(c, 6 + k))
    for k, c in enumerate(cfgs):
        _check(orc, sim, c, (k,))
    sim.close()
