"""Step parity in the default layout (no tile, interval or chunk asked for) of boxes
with an open end or a wall: 2D and 3D moving windows, r-z walls, r-z with a
window, in extents that leave ragged tiles or none that fits the LDS twice on a
CU; and of boxes whose only tiles are as large as that (a tile partly asked for,
a long interval)."""
import numpy as np
import pytest

from parity import F_TOL, J_TOL, MOM_TOL, POS_TOL, step_parity
from test_gpu_rz import _ring_plasma, _rz_fields, rz_step_parity
from test_gpu_window import _plasma, window_step_parity

pytestmark = pytest.mark.gpu


def _pic():
    from paper_1503_00276_amd import pic

    return pic


def _check(err, w_tol):
    assert err["pos"] <= POS_TOL and err["mom"] <= MOM_TOL and err["w"] <= w_tol, err
    assert err["J"] <= J_TOL and err["E"] <= F_TOL and err["B"] <= F_TOL, err


WINDOWS = [
    # nx, order, ppc, inject_ppc, extra
    ((37, 23), 2, 4, (2, 2), {}),
    ((53, 7), 1, 3, (3, 1), {"deposit": 1}),
    ((29, 31), 3, 3, (2, 2), {"accumulator": 2}),
    ((130, 66), 2, 6, (2, 2), {"inject_uth": 0.05, "inject_seed": 11}),
    ((33, 22, 17), 2, 1, (1, 1, 1), {}),          # no tile fits the LDS twice
    ((26, 14, 13), 3, 2, (1, 2, 1), {}),
    ((17, 12, 9), 1, 2, (1, 2, 1), {"deposit": 1}),
    ((16, 13, 11), 2, 2, (2, 1, 1), {"inject_uth": 0.1, "inject_seed": 3}),
]


@pytest.mark.parametrize("case", WINDOWS, ids=lambda c: "x".join(map(str, c[0])) + f"_o{c[1]}")
def test_window(orc, case):
    pic = _pic()
    nx, order, ppc, ippc, extra = case
    dim = len(nx)
    dx = (0.2, 0.23, 0.25)[:dim]
    x, u, w = _plasma(dim, nx, dx, ppc, 0.3, 5 + order)
    cfg = pic.Config(ndim=dim, nx=nx, dx=dx, dt=0.1 if dim == 2 else 0.08, shape_order=order, ion_density=1.0,
                     move_window=1, inject_ppc=ippc + (1,) * (3 - dim), inject_w=-1.0 / int(np.prod(ippc)), **extra)
    sim = pic.Pic(cfg)
    sim.load_particles(x, u, w, rqm=-1.0)
    i = sim.info()
    print("window", case, "tile", list(i.tile), "chunk", i.chunk, flush=True)
    E, B = np.random.default_rng(9).normal(0, 0.05, (2, 3, int(np.prod(nx))))
    sim.load_fields(E, B)
    shifts = removed = 0
    for n in range(6):
        err = window_step_parity(orc, sim, cfg, n, nload=len(x))
        assert err["inside"]
        _check(err, 1e-7)
        shifts += err["shift"]
        removed += err["removed"]
    assert shifts >= 2 and removed > 0
    sim.close()


@pytest.mark.parametrize("nx,order,extra", [((31, 23), 2, {}), ((67, 19), 1, {"deposit": 1}),
                                            ((24, 37), 3, {"accumulator": 2})],
                         ids=["31x23_o2", "67x19_o1", "24x37_o3"])
@pytest.mark.parametrize("window", [False, True])
def test_rz(orc, nx, order, extra, window):
    pic = _pic()
    dx = (0.2, 0.25)
    x, u, w = _ring_plasma(nx[0], nx[1], dx[0], dx[1], 3, 0.3, 60 + order)
    kw = dict(extra)
    if window:
        kw.update(move_window=1, inject_ppc=(2, 2, 1), inject_w=-0.2)
    cfg = pic.Config(ndim=2, nx=nx, dx=dx, dt=0.1, shape_order=order, geometry=pic.PIC_GEOM_RZ, ion_density=1.0, **kw)
    sim = pic.Pic(cfg)
    sim.load_particles(x, u, w, rqm=-1.0)
    i = sim.info()
    print("r-z", nx, order, window, "tile", list(i.tile), "chunk", i.chunk, flush=True)
    sim.load_fields(*_rz_fields(nx[0], nx[1], 13))
    removed = 0
    for n in range(5):
        err = window_step_parity(orc, sim, cfg, n, nload=len(x)) if window else rz_step_parity(orc, sim, cfg)
        _check(err, 1e-6)
        removed += err["removed"]
    assert removed > 0
    sim.close()


@pytest.mark.parametrize("nx,order,kw", [
    ((48, 16, 16), 2, {"tile": (48, 0, 0)}),
    ((25, 272), 3, {"tile": (0, 272)}),
    ((64, 128), 2, {"tile": (0, 64), "sort_interval": 12, "chunk": 2048}),
    ((42, 116), 2, {"sort_interval": 40}),
], ids=["48x16x16", "25x272", "64x128", "42x116"])
def test_large_tiles(orc, nx, order, kw):
    pic = _pic()
    dim = len(nx)
    dx = (0.2,) * dim
    cfg = pic.Config(ndim=dim, nx=nx, dx=dx, dt=0.7 * 0.2 / np.sqrt(dim), shape_order=order, ion_density=1.0, **kw)
    sim = pic.Pic(cfg)
    sim.load_particles(*_plasma(dim, nx, dx, 2, 0.3, 8), rqm=-1.0)
    i = sim.info()
    print("large tiles", nx, "tile", list(i.tile), "lds", i.lds_bytes, flush=True)
    for k in range(13):
        err = step_parity(orc, sim, cfg)
        assert err["pos"] <= POS_TOL and err["mom"] <= MOM_TOL, (k, err)
        assert err["J"] <= J_TOL and err["E"] <= F_TOL and err["B"] <= F_TOL, (k, err)
    sim.close()
