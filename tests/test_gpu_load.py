"""Loading particles on the GPU against the same conversion in numpy, bit for
bit: wrapped positions, offsets that round up to the next cell, several loads
into one species (in place, and growing it), several species, host arrays and
device tensors (also ones that are not contiguous FP64), a cell of more
particles than the interleaved ranks, windows in flight and r-z rows; what is
refused, and that a refused load changes nothing."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _pic():
    from paper_1503_00276_amd import pic

    return pic


def _stored(x, nx, dx, xmin):
    """The exported position of a loaded one: cell + FP32 offset, scaled."""
    out = np.empty_like(x)
    for d in range(x.shape[1]):
        L = float(nx[d])
        xi = np.fmod((x[:, d] - xmin[d]) / dx[d], L)
        xi = np.where(xi < 0, xi + L, xi)
        xi = np.where(xi >= L, xi - L, xi)
        c = np.floor(xi)
        e = (xi - c).astype(np.float32)
        up = e >= 1.0
        c, e = np.where(up, c + 1, c), np.where(up, np.float32(0), e)
        c = np.where(c >= L, c - L, c)
        out[:, d] = xmin[d] + (c + e.astype(np.float64)) * dx[d]
    return out


def _check(sim, parts, nx, dx, xmin):
    x, u, w = sim.state()
    np.testing.assert_array_equal(x, np.concatenate([_stored(p[0], nx, dx, xmin) for p in parts]))
    np.testing.assert_array_equal(u, np.concatenate([p[1] for p in parts]).astype(np.float32))
    np.testing.assert_array_equal(w, np.concatenate([p[2] for p in parts]).astype(np.float32))


def _draw(rng, n, nx, dx, xmin, spread=3.0):
    L = np.asarray(nx) * np.asarray(dx)
    x = np.asarray(xmin[:len(nx)]) + rng.uniform(-spread, 1 + spread, (n, len(nx))) * L
    return x, rng.normal(0, 0.3, (n, 3)), rng.uniform(-1, -0.1, n)


CASES = [
    # nx, tile, order
    ((20, 18), (0, 0), 2),
    ((37, 23), (8, 8), 1),
    ((300, 40), (30, 20), 3),
    ((9, 11, 8), (0, 0, 0), 2),
    ((16, 8, 12), (4, 4, 4), 3),
]


@pytest.mark.parametrize("device", [False, True])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c[0])))
def test_loads_match_the_conversion_bitwise(case, device):
    import torch

    pic = _pic()
    nx, tile, order = case
    dim = len(nx)
    dx, xmin = (0.1, 0.23, 0.31)[:dim], (-0.7, 1.3, 0.05)
    rng = np.random.default_rng(sum(nx))
    cfg = pic.Config(ndim=dim, nx=nx, dx=dx, xmin=xmin, dt=0.05, shape_order=order, tile=tile, sort_interval=1)
    sim = pic.Pic(cfg)
    a = _draw(rng, 1500, nx, dx, xmin)
    # on faces, a hair below them (the offset rounds up), and the box's ends
    k = rng.integers(0, np.asarray(nx), (200, dim))
    a[0][:200] = np.asarray(xmin[:dim]) + (k - 1e-9 * (rng.random((200, dim)) < 0.5)) * np.asarray(dx)
    a[0][200] = np.asarray(xmin[:dim])
    a[0][201] = np.asarray(xmin[:dim]) + np.asarray(nx) * np.asarray(dx)
    b = _draw(rng, 700, nx, dx, xmin, 0.0)     # grows the species
    b[0][:] = b[0][0]                          # more in one cell than the interleaved ranks
    c = _draw(rng, 3, nx, dx, xmin)
    other = _draw(rng, 900, nx, dx, xmin)

    def load(p, **kw):
        if device:
            t = [torch.tensor(v, device="cuda") for v in p]
            t[1] = t[1].t().contiguous().t()   # strided
            sim.load_particles(*t, **kw)
        else:
            sim.load_particles(*p, **kw)

    print("load", case, device, flush=True)
    load(a, rqm=-1.0)
    _check(sim, [a], nx, dx, xmin)
    load(other, rqm=4.0, species=3)
    load(b, rqm=-1.0)
    load(c, rqm=-1.0)
    _check(sim, [a, b, c, other], nx, dx, xmin)
    sim.step(3)
    sim.sync()
    assert sim.counts()[1] == 3103
    sim.close()


def test_append_in_place_within_the_capacity():
    pic = _pic()
    nx, dx, xmin = (24, 20), (0.2, 0.2), (0.0, 0.0, 0.0)
    rng = np.random.default_rng(4)
    cfg = pic.Config(ndim=2, nx=nx, dx=dx, dt=0.1, shape_order=1, capacity=3000)
    sim = pic.Pic(cfg)
    parts = [_draw(rng, 1000, nx, dx, xmin) for _ in range(3)]
    for k, p in enumerate(parts):
        sim.load_particles(*p, rqm=-1.0)
        _check(sim, parts[:k + 1], nx, dx, xmin)
    with pytest.raises(pic.PicError) as e:
        sim.load_particles(*_draw(rng, 1, nx, dx, xmin), rqm=-1.0)
    assert e.value.code == pic.PIC_E_NOMEM
    _check(sim, parts, nx, dx, xmin)
    sim.close()


@pytest.mark.parametrize("which,what", [(0, "position"), (1, "momentum"), (2, "weight")])
@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf])
def test_non_finite_input_is_refused_and_changes_nothing(which, what, value):
    pic = _pic()
    nx, dx, xmin = (16, 12), (0.2, 0.2), (0.0, 0.0, 0.0)
    rng = np.random.default_rng(5)
    sim = pic.Pic(pic.Config(ndim=2, nx=nx, dx=dx, dt=0.1, shape_order=2))
    good = _draw(rng, 400, nx, dx, xmin)
    sim.load_particles(*good, rqm=-1.0)
    bad = _draw(rng, 300, nx, dx, xmin)
    for k in range(which, 3):
        bad[k].reshape(-1)[-1] = value  # the first kind in order is reported
    with pytest.raises(pic.PicError) as e:
        sim.load_particles(*bad, rqm=-1.0)
    assert e.value.code == pic.PIC_E_RANGE and what in str(e.value)
    _check(sim, [good], nx, dx, xmin)
    sim.close()


def test_window_and_wall_ranges():
    pic = _pic()
    nz, nr, dz, dr = 24, 16, 0.2, 0.2
    cfg = pic.Config(ndim=2, nx=(nz, nr), dx=(dz, dr), dt=0.1, shape_order=1, move_window=1, inject_ppc=(1, 2, 1),
                     inject_w=-0.5, geometry=pic.PIC_GEOM_RZ)
    sim = pic.Pic(cfg)
    rng = np.random.default_rng(6)
    n = 500
    x = np.stack([rng.random(n) * nz * dz, rng.random(n) * (nr - 0.5) * dr * 0.999], 1)
    u, w = rng.normal(0, 0.1, (n, 3)), np.full(n, -0.2)
    sim.load_particles(x, u, w, rqm=-1.0)
    xs, _, _ = sim.state()
    # r-z: the cell coordinate is r/dr + 1/2
    cz, cr = x[:, 0] / dz, x[:, 1] / dr + 0.5
    np.testing.assert_array_equal(xs[:, 0], (np.floor(cz) + (cz - np.floor(cz)).astype(np.float32)) * dz)
    np.testing.assert_array_equal(xs[:, 1], (np.floor(cr) + (cr - np.floor(cr)).astype(np.float32) - 0.5) * dr)
    sim.step(9)  # four shifts
    sim.sync()
    x0 = 4 * dz
    for pos, text in [((x0 - 1e-6, 0.3), "window"), ((x0 + nz * dz, 0.3), "window"), ((x0 + 1.0, -1e-9), "radius"),
                      ((x0 + 1.0, (nr - 0.5) * dr), "radius"), ((x0 - 1.0, -1.0), "window")]:
        with pytest.raises(pic.PicError) as e:
            sim.load_particles(np.array([pos]), np.zeros((1, 3)), np.ones(1), rqm=-1.0)
        assert e.value.code == pic.PIC_E_RANGE and text in str(e.value), (pos, str(e.value))
    before = sim.state()
    new = np.array([[x0 + 1e-3, 0.25], [x0 + nz * dz - 1e-3, 2.0]])
    sim.load_particles(new, np.zeros((2, 3)), np.full(2, 0.3), rqm=-1.0)
    after = sim.state()
    for p, q in zip(before, after):
        np.testing.assert_array_equal(p, q[:-2])
    assert np.abs(after[0][-2:] - new).max() < 1e-6 and np.all(after[2][-2:] == np.float32(0.3))
    sim.load_particles(new, np.zeros((2, 3)), np.full(2, 0.1), rqm=1.0, species=1)
    sim.step(4)
    sim.sync()
    sim.close()
