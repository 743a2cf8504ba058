"""The one-phase kernels' unit of a step while the plasma speeds up from rest:
the bound on |u| that the unit follows has to rise at every step, also where
steps come one at a time, in whole captured cycles and in what is left of
them, for every species of the launch; and a load between two steps (of either
parity) keeps it.  A bound left behind would let a node's contributions pass
the int32 range and break the continuity equation: (rho1 - rho0)/dt + div J,
with rho from the stored positions, stays below 1e-4 of max |rho1 - rho0|/dt.
Each node's current carries a relative error of a few tens of FP32 roundings
(the factored shape differences, the weights, the unit), below 2^-18, and the
divergence of particles at one point sums 2 dim of them of like size; the
positions that rho is made of are rounded to half an ulp of the offset
(2^-25 of a cell) each step, against a move of at least 5e-3 of a cell in the
steps that are compared: 6e-6 of the change."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ndim,deposit,interval", [(2, 1, 1), (2, 1, 3), (2, 0, 2), (3, 1, 2)])
def test_unit_follows_a_plasma_accelerated_from_rest(ndim, deposit, interval):
    from paper_1503_00276_amd import pic

    n, dt = 1500, 0.05
    x = np.tile((np.full(ndim, 5) + 0.7) * 0.2, (n, 1))
    cfg = pic.Config(ndim=ndim, nx=(12,) * ndim, dx=(0.2,) * ndim, dt=dt, shape_order=1, tile=(6,) * ndim,
                     deposit=deposit, sort_interval=interval, chunk=2048, e0=(0.5, 0.3, 0.1))
    sim = pic.Pic(cfg)
    sim.load_particles(x, np.zeros((n, 3)), np.full(n, -0.37), rqm=-1.0)
    sim.load_particles(x + 0.4, np.zeros((n, 3)), np.full(n, 0.21), rqm=2.0, species=1)

    def check(label):
        print("step units", ndim, deposit, interval, label, flush=True)
        sim.rho_snapshot()
        rho0 = sim.rho()
        sim.step(1)
        rate = np.abs(sim.rho() - rho0).max() / dt
        assert rate > 0
        assert np.abs(sim.charge_residual()).max() <= 1e-4 * rate

    for steps in (2, 1, 4, 7):
        sim.step(steps)
        check(steps)
    # one more particle at rest: the bound of the others stays
    sim.load_particles(x[:1], np.zeros((1, 3)), np.full(1, -0.37), rqm=-1.0)
    check("after a load")
    sim.close()
