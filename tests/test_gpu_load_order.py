"""The default tile of a periodic 3D box does not depend on how its particles
are loaded: in one load, in slices, bunch or plasma first, in two species, after
an empty load or a refused one.  With the int64 current the tiling changes no
arithmetic, so the steps agree bit for bit too (particles by load order)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

NX, DX, PPC = (24, 20, 16), (0.2, 0.2, 0.2), 8


def _pic():
    from paper_1503_00276_amd import pic

    return pic


def _sim(pic, **kw):
    kw.setdefault("accumulator", pic.PIC_ACC_FIXED64)
    return pic.Pic(pic.Config(ndim=3, nx=NX, dx=DX, dt=0.1, shape_order=2, ion_density=1.0, **kw))


def _parts():
    rng = np.random.default_rng(11)
    L = np.asarray(NX) * np.asarray(DX)
    n = PPC * int(np.prod(NX))
    plasma = rng.random((n, 3)) * L, rng.normal(0, 0.2, (n, 3)), np.full(n, -1.0 / PPC)
    m = n // 32
    x = 0.5 * L + rng.normal(0, 0.3, (m, 3))
    u = rng.normal(0, 0.1, (m, 3))
    u[:, 0] += 20.0
    return plasma, (x, u, np.full(m, -0.25))


def _slices(p, k):
    return [tuple(a[i] for a in p) for i in np.array_split(np.arange(len(p[2])), k)]


def _result(sim):
    sim.step(3)
    out = (list(sim.info().tile), sim.fields(), sim.current(), sim.state())
    sim.close()
    return out


def _equal(a, b):
    """Tiles and grids; particles as a set (the loads order them differently)."""
    assert a[0] == b[0]
    for p, q in zip((*a[1], a[2]), (*b[1], b[2])):
        np.testing.assert_array_equal(p, q)
    rows = [np.concatenate([s[0], s[1], s[2][:, None]], 1) for s in (a[3], b[3])]
    rows = [r[np.lexsort(r.T)] for r in rows]
    np.testing.assert_array_equal(*rows)


def _one_load(pic):
    plasma, bunch = _parts()
    sim = _sim(pic)
    sim.load_particles(*(np.concatenate(z) for z in zip(plasma, bunch)), rqm=-1.0)
    return _result(sim)


@pytest.mark.parametrize("how", ["plasma first", "bunch first", "slices", "empty first", "refused first",
                                 "two species"])
def test_the_order_of_loads_does_not_matter(how):
    pic = _pic()
    plasma, bunch = _parts()
    print("load order", how, flush=True)
    sim = _sim(pic)
    loads = [plasma, bunch]
    if how == "bunch first":
        loads = [bunch, plasma]
    elif how == "slices":
        loads = _slices(plasma, 8) + _slices(bunch, 2)
    elif how == "empty first":
        sim.load_particles(np.zeros((0, 3)), np.zeros((0, 3)), np.zeros(0), rqm=-1.0)
    elif how == "refused first":
        for k in range(3):
            bad = [a[:1].copy() for a in plasma]
            bad[k].reshape(-1)[0] = np.nan
            with pytest.raises(pic.PicError):
                sim.load_particles(*bad, rqm=-1.0)
    for k, p in enumerate(loads):
        sim.load_particles(*p, rqm=-1.0, species=k if how == "two species" else 0)
    got, ref = _result(sim), _one_load(pic)
    _equal(got, ref)
    assert got[0] == [4, 4, 4]  # 512 particles a tile, at the box's 8.25 a cell
    if how == "bunch first":  # (alone it is a box of 0.25 a cell)
        sim = _sim(pic)
        sim.load_particles(*bunch, rqm=-1.0)
        assert int(np.prod(_result(sim)[0])) > 128


def test_a_refused_load_leaves_the_tile():
    pic = _pic()
    plasma, _ = _parts()
    tile = {}
    for how in ("good", "nan", "capacity"):
        sim = _sim(pic, capacity=len(plasma[2]))
        before = list(sim.info().tile)
        if how == "nan":
            with pytest.raises(pic.PicError):
                sim.load_particles(plasma[0][:1] * np.nan, plasma[1][:1], plasma[2][:1], rqm=-1.0)
        elif how == "capacity":
            with pytest.raises(pic.PicError):
                sim.load_particles(*(np.concatenate([a, a]) for a in plasma), rqm=-1.0)
        assert list(sim.info().tile) == before
        sim.load_particles(*plasma, rqm=-1.0)
        tile[how] = list(sim.info().tile)
        sim.close()
    assert tile["nan"] == tile["good"] and tile["capacity"] == tile["good"]


def test_a_tile_in_use_stays():
    """Loads after the first step with particles keep the tile; steps without
    particles settle nothing; the diagnostics before the first step see what
    is loaded."""
    pic = _pic()
    plasma, bunch = _parts()
    sim = _sim(pic)
    sim.step(2)
    sim.load_particles(*bunch, rqm=-1.0)
    rho = sim.rho()
    sim.load_particles(*plasma, rqm=-1.0)
    assert np.abs(sim.rho() - rho).max() > 0.1
    x, u, w = sim.state()
    np.testing.assert_array_equal(u[:len(bunch[1])], bunch[1].astype(np.float32))
    sim.step(1)
    tile = list(sim.info().tile)
    assert tile == [4, 4, 4]
    sim.close()
    sim = _sim(pic)
    sim.load_particles(*bunch, rqm=-1.0)
    sim.step(1)
    tile = list(sim.info().tile)
    sim.load_particles(*plasma, rqm=-1.0)
    sim.step(1)
    assert list(sim.info().tile) == tile
    assert sim.counts()[1] == len(bunch[2]) + len(plasma[2])
    sim.close()


def test_parity_after_the_stores_moved(orc):
    from parity import F_TOL, J_TOL, MOM_TOL, POS_TOL, step_parity

    pic = _pic()
    plasma, bunch = _parts()
    sim = _sim(pic, accumulator=0)
    sim.load_particles(*bunch, rqm=-1.0)
    sim.load_particles(*plasma, rqm=-1.0)
    for k in range(2):
        err = step_parity(orc, sim, sim.cfg)
        assert err["pos"] <= POS_TOL and err["mom"] <= MOM_TOL, (k, err)
        assert err["J"] <= J_TOL and err["E"] <= F_TOL and err["B"] <= F_TOL, (k, err)
    sim.close()
