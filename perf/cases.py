"""Performance cases of the particle-in-cell step library.

Each case is a plain dict of values.  ``prepare`` makes what a program holds
before the call (device tensors and a loaded simulation), ``run`` makes one
pass through the public binding (``paper_1503_00276_amd.pic``), ``work`` counts
what one pass cannot do without, and ``exact`` computes the same outputs in
64 bits with plain torch.

Kinds of plasma (``plasma``): ``thermal`` (Maxwellian electrons at random
positions over fixed ions), ``laser`` (a laser pulse in a cold, slightly warm
plasma on a lattice), ``beam`` (a relativistic electron bunch in a cold
lattice plasma).  Kinds of pass (``call``):

  step   n steps of a loaded simulation, then what ``out`` names
  run    a whole short run: create, load, n steps, then the final state
  batch  n steps of a batch of 2D instances, then every instance's grids
  dump   no steps: the diagnostics and exports of a dump
"""
import math

import numpy as np
import torch

from paper_1503_00276_amd import pic

DEV = "cuda:0"


# --------------------------------------------------------------------------
# the cases
# --------------------------------------------------------------------------

def _case(name, **kw):
    c = dict(call="step", plasma="thermal", dim=2, n0=64, n1=64, n2=1, order=1, ppc=8, uth=0.02, steps=10,
             out="grids", accumulator=0, deposit=0, smooth=0, window=0, rz=0, instances=0)
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # a small thermal box probed after every step (time histories of the
        # energy and the fields): the smallest call, latency and launches
        _case("thermal2d_probe", n0=64, n1=64, order=1, ppc=16, uth=0.01, steps=1, out="probe"),
        # one member of a parameter scan from nothing to its final state: the
        # 64x64 thermal box, created, loaded, 100 steps, exported
        _case("thermal2d_whole_run", call="run", n0=64, n1=64, order=1, ppc=16, uth=0.01, steps=100),
        # the 2D laser wakefield in a periodic box, quadratic shape: the
        # ordinary 2D run between two grid dumps
        _case("laser2d", plasma="laser", n0=1024, n1=256, order=2, ppc=8, uth=0.005, steps=100),
        # the same with the window that moves at c: particles leave and enter
        # at every step
        _case("laser2d_window", plasma="laser", n0=768, n1=192, order=2, ppc=8, uth=0.005, steps=50, window=1),
        # reproducible int64 current, cubic shape, smoothed current, a ragged
        # grid: a 2D study that needs bitwise repeatable, low-noise currents
        _case("thermal2d_smooth_fixed", n0=300, n1=200, order=3, ppc=9, uth=0.05, steps=40, accumulator=2, smooth=3),
        # the Villasenor-Buneman deposit of the dissertation's deck
        _case("tristan2d", n0=250, n1=170, order=1, ppc=12, uth=0.1, steps=50, deposit=1),
        # 3D beam-driven wake, quadratic shape
        _case("beam3d", plasma="beam", dim=3, n0=128, n1=64, n2=64, order=2, ppc=8, uth=0.002, steps=40),
        # the large 3D box, cubic shape, between two density dumps
        _case("cubic3d", dim=3, n0=256, n1=128, n2=128, order=3, ppc=4, uth=0.02, steps=20, out="density"),
        # an odd-sized 3D box, linear shape
        _case("linear3d_odd", dim=3, n0=45, n1=37, n2=53, order=1, ppc=6, uth=0.1, steps=25),
        # beam-driven wake in r-z with the window along z, two species
        _case("beam_rz_window", plasma="beam", n0=384, n1=96, order=2, ppc=4, uth=0.0, steps=50, window=1, rz=1),
        # a parameter scan of uneven boxes advanced together
        _case("scan_batch", call="batch", instances=24, uth=0.02, steps=25),
        # everything a dump writes: charge density, Gauss residual, energies,
        # fields, current and the particles
        _case("dump3d", call="dump", dim=3, n0=64, n1=64, n2=48, order=2, ppc=6, uth=0.05, steps=0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["small", "flat", "flat", "laser", "window", "box", "box", "beam", "rz", "batch", "run", "dump"])
    uth = round(math.exp(rng.uniform(math.log(0.005), math.log(0.2))), 4)
    if kind == "small":
        return _case("", n0=_log_int(rng, 24, 128), n1=_log_int(rng, 24, 128), order=rng.randint(1, 3),
                     ppc=rng.randint(2, 20), uth=uth, steps=rng.randint(1, 3), out="probe")
    if kind == "flat":
        order = rng.randint(1, 3)
        return _case("", n0=_log_int(rng, 96, 1024), n1=_log_int(rng, 64, 300), order=order, ppc=rng.randint(2, 12),
                     uth=uth, steps=rng.randint(20, 60), accumulator=rng.choice([0, 0, 2]),
                     smooth=rng.choice([0, 0, 2, 4]), deposit=1 if order == 1 and rng.random() < 0.4 else 0)
    if kind == "laser":
        return _case("", plasma="laser", n0=_log_int(rng, 760, 1200), n1=_log_int(rng, 64, 256),
                     order=rng.randint(1, 3), ppc=rng.choice([4, 8]), uth=0.005, steps=rng.randint(40, 100))
    if kind == "window":
        return _case("", plasma="laser", n0=_log_int(rng, 760, 1000), n1=_log_int(rng, 48, 200),
                     order=rng.randint(1, 3), ppc=rng.choice([4, 8]), uth=0.005, steps=rng.randint(20, 50), window=1)
    if kind == "box":
        return _case("", dim=3, n0=_log_int(rng, 24, 160), n1=_log_int(rng, 24, 96), n2=_log_int(rng, 24, 96),
                     order=rng.randint(1, 3), ppc=rng.randint(1, 8), uth=uth, steps=rng.randint(8, 20),
                     out=rng.choice(["grids", "density"]))
    if kind == "beam":
        return _case("", plasma="beam", dim=3, n0=_log_int(rng, 96, 160), n1=_log_int(rng, 32, 64),
                     n2=_log_int(rng, 32, 64), order=rng.randint(1, 3), ppc=8, uth=0.002, steps=rng.randint(12, 40))
    if kind == "rz":
        return _case("", plasma="beam", n0=_log_int(rng, 128, 500), n1=_log_int(rng, 32, 120),
                     order=rng.randint(1, 3), ppc=4, uth=0.0, steps=rng.randint(20, 50), window=rng.randint(0, 1), rz=1)
    if kind == "batch":
        return _case("", call="batch", instances=rng.randint(3, 24), uth=uth, steps=rng.randint(10, 25))
    if kind == "run":
        return _case("", call="run", n0=_log_int(rng, 32, 128), n1=_log_int(rng, 32, 128), order=rng.randint(1, 3),
                     ppc=rng.randint(4, 16), uth=min(uth, 0.05), steps=rng.randint(30, 100))
    dim = rng.randint(2, 3)
    return _case("", call="dump", dim=dim, n0=_log_int(rng, 32, 64) * (1 if dim == 3 else 6),
                 n1=_log_int(rng, 32, 64) * (1 if dim == 3 else 3), n2=_log_int(rng, 24, 48) if dim == 3 else 1,
                 order=rng.randint(1, 3), ppc=rng.randint(2, 6), uth=uth, steps=0)


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _rand(g, *shape):
    return torch.rand(*shape, dtype=torch.float64, device=DEV, generator=g)


def _randn(g, *shape):
    return torch.randn(*shape, dtype=torch.float64, device=DEV, generator=g)


def _cells(nx):
    """[ncell, dim] integer cell coordinates, axis 1 fastest."""
    ax = [torch.arange(n, dtype=torch.float64, device=DEV) for n in reversed(nx)]
    m = torch.meshgrid(*ax, indexing="ij")
    return torch.stack([t.reshape(-1) for t in reversed(m)], 1)


def _sub(per_axis):
    """Regular sub-lattice offsets of a cell, [prod, dim]."""
    return (_cells(per_axis) + 0.5) / torch.tensor(per_axis, dtype=torch.float64, device=DEV)


def _lattice(nx, per_axis):
    """Lattice positions in cell units."""
    return (_cells(nx)[:, None, :] + _sub(per_axis)[None]).reshape(-1, len(nx))


def _per_axis(ppc, dim):
    return {(8, 3): (2, 2, 2), (8, 2): (2, 4), (4, 2): (2, 2)}[(ppc, dim)]


def _spec(case):
    """Cell sizes, time step and the library's configuration of a case."""
    dim = case["dim"]
    nx = (case["n0"], case["n1"], case["n2"])[:dim]
    if case["plasma"] == "laser":
        dx = (0.05, 0.2)
        dt = 0.95 / math.sqrt(sum(1.0 / d ** 2 for d in dx))
        ion = 0.01
    elif dim == 3 or case["rz"]:
        dx, dt, ion = (0.05,) * dim, 0.02, 1.0
    else:
        dx, dt, ion = (0.2, 0.2), 0.1, 1.0
    kw = {}
    if case["smooth"]:
        # binomial passes and a compensator along every axis
        kw["smooth"] = ([(1.0, 2.0, 1.0)] * (case["smooth"] - 1) + [(-1.0, 6.0, -1.0)],) * dim
    if case["window"]:
        pa = _per_axis(case["ppc"], dim)
        # room for what the pulse sweeps up in front of it
        kw.update(move_window=1, inject_ppc=pa + (1,) * (3 - dim), inject_w=-ion / case["ppc"],
                  capacity=int(1.5 * case["ppc"] * math.prod(nx)) + 4096)
    if case["rz"]:
        kw["geometry"] = pic.PIC_GEOM_RZ
    cfg = pic.Config(ndim=dim, nx=nx, dx=dx, dt=dt, shape_order=case["order"], ion_density=ion,
                     accumulator=case["accumulator"], deposit=case["deposit"], **kw)
    return cfg


def _inputs(case, seed):
    """[(x, u, w)] per species (device tensors) and (E, B) or None."""
    cfg, g = _spec(case), _gen(seed)
    nx, dim, ppc = tuple(cfg.nx), case["dim"], case["ppc"]
    dx = torch.tensor(cfg.dx[:dim], dtype=torch.float64, device=DEV)
    fields = None
    if case["plasma"] == "thermal":
        c = _cells(nx).repeat_interleave(ppc, 0)
        x = (c + _rand(g, *c.shape)) * dx
        u = _randn(g, len(x), 3) * case["uth"]
        w = torch.full((len(x),), -cfg.ion_density / ppc, dtype=torch.float64, device=DEV)
        return cfg, [(x, u, w)], None
    if case["plasma"] == "laser":
        x = _lattice(nx, _per_axis(ppc, 2)) * dx
        u = _randn(g, len(x), 3) * case["uth"]
        w = torch.full((len(x),), -cfg.ion_density / ppc, dtype=torch.float64, device=DEV)
        # polynomial rise and fall over 30/k0 in all, Gaussian across, a0 = 2 (+-5 %)
        a0 = 2.0 * (1.0 + 0.05 * (2.0 * float(_rand(g, 1)) - 1.0))
        E = torch.zeros(3, nx[1], nx[0], dtype=torch.float64, device=DEV)
        B = torch.zeros_like(E)
        i = torch.arange(nx[0], dtype=torch.float64, device=DEV)
        j = torch.arange(nx[1], dtype=torch.float64, device=DEV)
        x0, half = (nx[0] * cfg.dx[0]) - 32.0, 15.0
        tr = torch.exp(-(((j + 0.5) * cfg.dx[1] - 0.5 * nx[1] * cfg.dx[1]) / (20 * math.pi)) ** 2)

        def wave(x1):
            xi = x1 - x0
            s = torch.clamp(torch.minimum(xi, 30.0 - xi) / half, 0.0, 1.0)
            return a0 * (10 * s ** 3 - 15 * s ** 4 + 6 * s ** 5) * torch.sin(x1)

        E[1] = tr[:, None] * wave(i * cfg.dx[0])[None]
        B[2] = tr[:, None] * wave((i + 0.5) * cfg.dx[0])[None]
        return cfg, [(x, u, w)], (E.reshape(3, -1).contiguous(), B.reshape(3, -1).contiguous())
    # beam: lattice background and a bi-Gaussian bunch, gamma 2e4 (0.1 % spread)
    ncell = cfg.ncell
    nb = max(256, ncell // (16 if dim == 2 else 4))
    L = [n * d for n, d in zip(nx, cfg.dx)]
    gam = 2.0e4 * (1.0 + 1.0e-3 * _randn(g, nb))
    ub = torch.zeros(nb, 3, dtype=torch.float64, device=DEV)
    ub[:, 0] = torch.sqrt(gam ** 2 - 1.0)
    zc, sz, sr, peak = 0.65 * L[0], 0.5, 0.1, 4.0
    if case["rz"]:
        # rings: weight proportional to the radius of the lattice point
        cc = _lattice(nx, _per_axis(ppc, 2))
        cc = cc[(cc[:, 1] >= 0.5) & (cc[:, 1] < nx[1] - 0.5)]
        r = cc[:, 1] - 0.5
        x = torch.stack([cc[:, 0], r], 1) * dx
        u = torch.zeros(len(x), 3, dtype=torch.float64, device=DEV)
        w = -r / ppc
        zb = torch.clamp(zc + sz * _randn(g, nb), 0.2 * L[0], 0.98 * L[0])
        rb = torch.clamp(sr * torch.sqrt(-2.0 * torch.log(1.0 - _rand(g, nb))), 0.0, 0.8 * (nx[1] - 0.5) * cfg.dx[1])
        # a ring of weight w holds the charge 2 pi dr^2 dz w
        q = peak * (2 * math.pi) ** 1.5 * sz * sr * sr / nb
        wb = torch.full((nb,), -q / (2 * math.pi * cfg.dx[1] ** 2 * cfg.dx[0]), dtype=torch.float64, device=DEV)
        return cfg, [(x, u, w), (torch.stack([zb, rb], 1), ub, wb)], None
    x = _lattice(nx, _per_axis(ppc, 3)) * dx
    u = _randn(g, len(x), 3) * case["uth"]
    w = torch.full((len(x),), -1.0 / ppc, dtype=torch.float64, device=DEV)
    ctr = torch.tensor([zc, 0.5 * L[1], 0.5 * L[2]], dtype=torch.float64, device=DEV)
    xb = _randn(g, nb, 3) * torch.tensor([sz, sr, sr], dtype=torch.float64, device=DEV) + ctr
    wb = torch.full((nb,), -peak * (2 * math.pi) ** 1.5 * sz * sr * sr / (nb * float(np.prod(cfg.dx))),
                    dtype=torch.float64, device=DEV)
    return cfg, [(torch.cat([x, xb]), torch.cat([u, ub]), torch.cat([w, wb]))], None


def _batch_inputs(case, seed):
    """Uneven 2D thermal boxes, linear or quadratic, as a parameter scan has them."""
    r = np.random.default_rng(1503 + case["instances"])  # the boxes belong to the case, their particles to the seed
    grids = [(64, 64), (128, 128), (256, 128), (512, 256)]
    out = []
    for k in range(case["instances"]):
        nx = grids[int(r.integers(0, 4))]
        c = _case("", n0=nx[0], n1=nx[1], order=int(r.integers(1, 3)), ppc=int(r.integers(4, 13)),
                  uth=case["uth"] * float(r.uniform(0.5, 1.5)))
        out.append(_inputs(c, seed * 1000 + k))
    return out


def _load(sim, species, fields):
    for s, (x, u, w) in enumerate(species):
        sim.load_particles(x, u, w, rqm=-1.0, species=s)
    if fields is not None:
        sim.load_fields(*fields)


def prepare(case, seed):
    if case["call"] == "batch":
        inst = _batch_inputs(case, seed)
        sim = pic.PicBatch([i[0] for i in inst])
        for k, (_, ((x, u, w),), _) in enumerate(inst):
            sim.load_particles(k, x, u, w, rqm=-1.0)
        return {"case": case, "sim": sim}
    cfg, species, fields = _inputs(case, seed)
    state = {"case": case, "cfg": cfg}
    if case["call"] == "run":
        state["inputs"] = (species, fields)
        return state
    sim = pic.Pic(cfg)
    _load(sim, species, fields)
    state["sim"] = sim
    if case["out"] == "density" or case["call"] == "dump":
        state["rho"] = torch.empty(cfg.ncell, dtype=torch.float64, device=DEV)
        state["gauss"] = torch.empty(cfg.ncell, dtype=torch.float64, device=DEV)
    if case["call"] == "dump":
        sim.load_fields(*_noise_fields(cfg, seed))
    return state


def _noise_fields(cfg, seed):
    g = _gen(seed + 77)
    return 0.05 * _randn(g, 3, cfg.ncell), 0.05 * _randn(g, 3, cfg.ncell)


# --------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------

def _f32(a):
    """Dumps hold the library's single-precision values."""
    return a.astype(np.float32)


def _grids(sim, *i):
    E, B = sim.fields(*i)
    return {"E": _f32(E), "B": _f32(B), "J": _f32(sim.current(*i))}


def run(state):
    case = state["case"]
    if case["call"] == "run":
        sim = pic.Pic(state["cfg"])
        _load(sim, *state["inputs"])
        sim.step(case["steps"])
        out = _grids(sim)
        x, u, w = sim.state()
        out.update(energy=_f32(sim.energy()), x=_f32(x), u=_f32(u), w=_f32(w))
        sim.close()
        return out
    sim = state["sim"]
    if case["call"] == "dump":
        out = _grids(sim)
        sim.diag_noalloc(pic.PIC_DIAG_RHO, state["rho"])
        sim.diag_noalloc(pic.PIC_DIAG_GAUSS_RESIDUAL, state["gauss"])
        x, u, w = sim.state()
        out.update(rho=state["rho"], gauss=state["gauss"], energy=sim.energy(), momentum=_f32(sim.momentum()),
                   x=x, u=u, w=w)
        return out
    sim.step(case["steps"])
    if case["call"] == "batch":
        return [np.concatenate([*sim.fields(k), sim.current(k)]).astype(np.float32) for k in range(case["instances"])]
    if case["out"] == "density":
        sim.diag_noalloc(pic.PIC_DIAG_RHO, state["rho"])
        return {"rho": state["rho"].float(), "energy": _f32(sim.energy())}
    out = _grids(sim)
    if case["out"] == "probe":
        out["energy"] = _f32(sim.energy())
    return out


# --------------------------------------------------------------------------
# what a pass cannot do without
# --------------------------------------------------------------------------

def work(case):
    if case["call"] == "batch":
        r = np.random.default_rng(1503 + case["instances"])
        grids = [(64, 64), (128, 128), (256, 128), (512, 256)]
        tot = {"bytes": 0.0, "flops": 0.0}
        for _ in range(case["instances"]):
            nx = grids[int(r.integers(0, 4))]
            c = _case("", n0=nx[0], n1=nx[1], order=int(r.integers(1, 3)), ppc=int(r.integers(4, 13)),
                      steps=case["steps"])
            r.uniform(0.5, 1.5)
            w = work(c)
            tot = {k: tot[k] + w[k] for k in tot}
        return tot
    d, o = case["dim"], case["order"]
    ncell = case["n0"] * case["n1"] * case["n2"]
    n = ncell * case["ppc"] + (max(256, ncell // (16 if d == 2 else 4)) if case["plasma"] == "beam" else 0)
    k = o + 1
    # per particle and step: its state read and written (cell, offsets, u; w
    # read); per cell: E, B read for the gather, J written, and the field
    # solve (E, B, J read, E, B written)
    by = case["steps"] * (n * (36 + 8 * d) + ncell * (24 + 12 + 36 + 24))
    # gather: six components of k^d taps; deposit: three components of about
    # (k-1) k^(d-1) nodes in 3D (2D: two of (k-1) k and one of k^2), three
    # operations each; push, moves and shapes
    taps = 6 * k ** d
    nodes = 3 * (k - 1) * k ** (d - 1) if d == 3 else 2 * (k - 1) * k + k * k
    fl = case["steps"] * (n * (2 * taps + 3 * nodes + 60 + 20 * d * k) + 60 * ncell)
    if case["call"] == "run":
        by += n * (d + 4) * 8 * 2  # inputs read, state written
    if case["call"] == "dump":
        by += n * (d + 4) * (4 + 8) + ncell * (36 + 72 + 16)
        fl += n * 2 * k ** d
    elif case["out"] == "density":
        by += n * (4 * d + 8) + ncell * 8
        fl += n * 2 * k ** d
    else:
        by += ncell * 9 * (4 + 4)
    return {"bytes": float(by), "flops": float(fl)}


# --------------------------------------------------------------------------
# the same in 64 bits
# --------------------------------------------------------------------------

def _spline(order, d):
    """B-spline of the given order at distance d (cells)."""
    a = d.abs()
    if order == 1:
        return torch.clamp(1.0 - a, min=0.0)
    if order == 2:
        return torch.where(a <= 0.5, 0.75 - a * a, 0.5 * torch.clamp(1.5 - a, min=0.0) ** 2)
    return torch.where(a <= 1.0, (4.0 - 6.0 * a * a + 3.0 * a ** 3) / 6.0, torch.clamp(2.0 - a, min=0.0) ** 3 / 6.0)


def _first(order, x):
    """First node of the shape of a particle at x (nodes at the integers)."""
    return torch.floor(x) - (1 if order == 3 else 0) if order != 2 else torch.floor(x + 0.5) - 1


class _Exact:
    """One periodic Cartesian plasma in 64 bits."""

    def __init__(self, cfg, species, fields, order):
        self.cfg, self.o, self.dim = cfg, order, cfg.ndim
        self.nx = [int(n) for n in cfg.nx[:cfg.ndim]]
        x, u, w = species
        self.dx = [float(d) for d in cfg.dx[:cfg.ndim]]
        # the library keeps single-precision momenta, weights and offsets
        self.x = [x[:, d] / self.dx[d] for d in range(self.dim)]
        self.u = [u[:, d].float().double() for d in range(3)]
        self.w = w.float().double()
        self.F = torch.zeros(6, cfg.ncell, dtype=torch.float64, device=DEV)
        if fields is not None:
            self.F[:3], self.F[3:] = fields[0].float().double(), fields[1].float().double()
        self.J = torch.zeros(3, cfg.ncell, dtype=torch.float64, device=DEV)

    def nodes(self, base, d, count):
        n = self.nx[d]
        stride = int(np.prod(self.nx[:d], dtype=np.int64)) if d else 1
        return [torch.remainder(base + k, n).long() * stride for k in range(count)]

    def gather(self):
        o, out = self.o, []
        per = []
        for d in range(self.dim):
            both = []
            for half in (0.0, 0.5):
                xs = self.x[d] - half
                b = _first(o, xs)
                both.append((self.nodes(b, d, o + 1), [_spline(o, xs - (b + k)) for k in range(o + 1)]))
            per.append(both)
        for c in range(6):
            acc = torch.zeros_like(self.w)
            st = [(c == d) if c < 3 else (c - 3 != d) for d in range(self.dim)]
            ax = [per[d][int(st[d])] for d in range(self.dim)]
            for k in range(o + 1 if self.dim == 3 else 1):
                for j in range(o + 1):
                    row, wt = ax[1][0][j], ax[1][1][j]
                    if self.dim == 3:
                        row, wt = row + ax[2][0][k], wt * ax[2][1][k]
                    for i in range(o + 1):
                        acc += self.F[c][ax[0][0][i] + row] * (wt * ax[0][1][i])
            out.append(acc)
        return out

    def curl(self, V, fwd):
        """Components of curl V with forward or backward differences."""
        shp = list(reversed(self.nx))
        V = [v.reshape(shp) for v in V]

        def D(v, d):
            if d >= self.dim:
                return torch.zeros_like(v)
            a = self.dim - 1 - d
            return ((torch.roll(v, -1, a) - v) if fwd else (v - torch.roll(v, 1, a))) / self.dx[d]

        return torch.stack([(D(V[2], 1) - D(V[1], 2)).reshape(-1), (D(V[0], 2) - D(V[2], 0)).reshape(-1),
                            (D(V[1], 0) - D(V[0], 1)).reshape(-1)])

    def smooth(self):
        shp = [3] + list(reversed(self.nx))
        J = self.J.reshape(shp)
        for d, passes in enumerate(self.cfg.smooth):
            a = self.dim - d
            for p in passes:
                s = sum(p)
                J = (p[0] * torch.roll(J, 1, a) + p[1] * J + p[2] * torch.roll(J, -1, a)) / s
        self.J = J.reshape(3, -1).contiguous()

    def step(self):
        o, dim, dt = self.o, self.dim, self.cfg.dt
        Ex, Ey, Ez, Bx, By, Bz = self.gather()
        h = -0.5 * dt  # charge-to-mass ratio -1
        m = [self.u[0] + h * Ex, self.u[1] + h * Ey, self.u[2] + h * Ez]
        gi = 1.0 / torch.sqrt(1.0 + m[0] ** 2 + m[1] ** 2 + m[2] ** 2)
        t = [h * Bx * gi, h * By * gi, h * Bz * gi]
        s = 2.0 / (1.0 + t[0] ** 2 + t[1] ** 2 + t[2] ** 2)
        p = [m[0] + m[1] * t[2] - m[2] * t[1], m[1] + m[2] * t[0] - m[0] * t[2], m[2] + m[0] * t[1] - m[1] * t[0]]
        self.u = [m[0] + s * (p[1] * t[2] - p[2] * t[1]) + h * Ex, m[1] + s * (p[2] * t[0] - p[0] * t[2]) + h * Ey,
                  m[2] + s * (p[0] * t[1] - p[1] * t[0]) + h * Ez]
        gi = 1.0 / torch.sqrt(1.0 + self.u[0] ** 2 + self.u[1] ** 2 + self.u[2] ** 2)
        new = [self.x[d] + dt * self.u[d] * gi / self.dx[d] for d in range(dim)]
        W = o + 2
        S, Dl, idx, P = [], [], [], []
        for d in range(dim):
            b = torch.minimum(_first(o, self.x[d]), _first(o, new[d]))
            s0 = [_spline(o, self.x[d] - (b + k)) for k in range(W)]
            dd = [_spline(o, new[d] - (b + k)) - s0[k] for k in range(W)]
            S.append(s0)
            Dl.append(dd)
            idx.append(self.nodes(b, d, W))
            acc, pr = torch.zeros_like(self.w), []
            for k in range(W - 1):
                acc = acc + dd[k]
                pr.append(-self.w * (self.dx[d] / dt) * acc)
            P.append(pr)
        self.J = torch.zeros_like(self.J)
        if dim == 2:
            v3 = self.w * self.u[2] * gi
            for j in range(W):
                for i in range(W):
                    at = idx[0][i] + idx[1][j]
                    if i < W - 1:
                        self.J[0].index_add_(0, at, P[0][i] * (S[1][j] + 0.5 * Dl[1][j]))
                    if j < W - 1:
                        self.J[1].index_add_(0, at, P[1][j] * (S[0][i] + 0.5 * Dl[0][i]))
                    self.J[2].index_add_(0, at, v3 * (S[0][i] * S[1][j] + 0.5 * (Dl[0][i] * S[1][j] + S[0][i] * Dl[1][j])
                                                      + Dl[0][i] * Dl[1][j] / 3.0))
        else:
            for A in range(3):
                Bq, C = (A + 1) % 3, (A + 2) % 3
                for c in range(W):
                    for b in range(W):
                        T = (S[Bq][b] * S[C][c] + 0.5 * (Dl[Bq][b] * S[C][c] + S[Bq][b] * Dl[C][c])
                             + Dl[Bq][b] * Dl[C][c] / 3.0)
                        at = idx[Bq][b] + idx[C][c]
                        for a in range(W - 1):
                            self.J[A].index_add_(0, idx[A][a] + at, P[A][a] * T)
        if self.cfg.smooth:
            self.smooth()
        self.x = [torch.remainder(new[d], self.nx[d]) for d in range(dim)]
        E, B = self.F[:3], self.F[3:]
        B = B - 0.5 * dt * self.curl(E, True)
        E = E + dt * (self.curl(B, False) - self.J)
        B = B - 0.5 * dt * self.curl(E, True)
        self.F = torch.cat([E, B])

    def rho(self):
        o = self.o
        rho = torch.full((self.cfg.ncell,), float(self.cfg.ion_density), dtype=torch.float64, device=DEV)
        per = []
        for d in range(self.dim):
            b = _first(o, self.x[d])
            per.append((self.nodes(b, d, o + 1), [_spline(o, self.x[d] - (b + k)) for k in range(o + 1)]))
        for k in range(o + 1 if self.dim == 3 else 1):
            for j in range(o + 1):
                row, wt = per[1][0][j], self.w * per[1][1][j]
                if self.dim == 3:
                    row, wt = row + per[2][0][k], wt * per[2][1][k]
                for i in range(o + 1):
                    rho.index_add_(0, per[0][0][i] + row, wt * per[0][1][i])
        return rho

    def div(self):
        shp = list(reversed(self.nx))
        out = torch.zeros(shp, dtype=torch.float64, device=DEV)
        for d in range(self.dim):
            v = self.F[d].reshape(shp)
            out += (v - torch.roll(v, 1, self.dim - 1 - d)) / self.dx[d]
        return out.reshape(-1)

    def energy(self):
        V = float(np.prod(self.dx))
        usq = self.u[0] ** 2 + self.u[1] ** 2 + self.u[2] ** 2
        e = [0.5 * V * float((self.F[:3] ** 2).sum()), 0.5 * V * float((self.F[3:] ** 2).sum()),
             V * float((-self.w * usq / (torch.sqrt(1.0 + usq) + 1.0)).sum())]
        return np.array(e + [sum(e)])

    def momentum(self):
        V = float(np.prod(self.dx))
        return np.array([V * float((-self.w * u).sum()) for u in self.u])

    def grids(self):
        return {"E": self.F[:3].cpu().numpy(), "B": self.F[3:].cpu().numpy(), "J": self.J.cpu().numpy()}

    def state(self):
        return {"x": torch.stack([x * d for x, d in zip(self.x, self.dx)], 1).cpu().numpy(),
                "u": torch.stack(self.u, 1).cpu().numpy(), "w": self.w.cpu().numpy()}


def exact(case, seed):
    if case["window"] or case["rz"] or case["deposit"]:
        return None  # no short 64-bit form of these boundaries and of the cut paths
    if case["call"] == "batch":
        out = []
        for cfg, (sp,), _ in _batch_inputs(case, seed):
            e = _Exact(cfg, sp, None, cfg.shape_order)
            for _ in range(case["steps"]):
                e.step()
            out.append(torch.cat([e.F, e.J]).cpu().numpy())
        return out
    cfg, species, fields = _inputs(case, seed)
    if case["call"] == "dump":
        fields = _noise_fields(cfg, seed)
    e = _Exact(cfg, species[0], fields, case["order"])
    for _ in range(case["steps"]):
        e.step()
    if case["call"] == "dump":
        out = e.grids()
        rho = e.rho()
        out.update(rho=rho, gauss=e.div() - rho, energy=e.energy(), momentum=e.momentum(), **e.state())
        return out
    if case["out"] == "density":
        return {"rho": e.rho(), "energy": e.energy()}
    out = e.grids()
    if case["call"] == "run":
        out.update(energy=e.energy(), **e.state())
    elif case["out"] == "probe":
        out["energy"] = e.energy()
    return out
