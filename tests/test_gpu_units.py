"""The 32-bit current tile's unit where its bound is tightest: a full work item
of particles at one point, all moving alike, so that the densest nodes sum
near-maximal contributions of one sign, at speeds from half the light's down
to a fraction of an ulp of the offset per step (there FP32 moves a particle by
a whole ulp, more than v dt).  An overflowing sum would break the continuity
equation: (rho1 - rho0)/dt + div J, with rho from the stored positions, stays
below 1e-4 of max |rho1 - rho0|/dt.  Each node's current carries a relative
error of at most a few tens of FP32 roundings (the factored shape differences,
the weights, the sum's unit of at most 2^-30 of the item's bound: 2^-18), and
the divergence of a plasma at one point sums 2 dim of them of like size:
below 2^-15."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

ULP = 2.0 ** -24  # of an offset in [1/2, 1)


@pytest.mark.parametrize("ndim,order", [(2, 1), (2, 2), (2, 3), (3, 1), (3, 2), (3, 3)])
@pytest.mark.parametrize("move", [0.4, 0.01, 20 * ULP, 0.6 * ULP])
def test_full_item_of_equal_particles_conserves_charge(ndim, order, move):
    from paper_1503_00276_amd import pic

    nx, dx, dt = (12,) * ndim, (0.2,) * ndim, 0.1
    n = 1024 if ndim == 2 else 768
    x = np.tile((np.full(ndim, 5) + 0.7) * 0.2, (n, 1))
    v = np.array([1.0, 0.5, 0.25]) * move * 0.2 / dt
    u = np.tile(v / np.sqrt(1.0 - v @ v), (n, 1))
    cfg = pic.Config(ndim=ndim, nx=nx, dx=dx, dt=dt, shape_order=order, tile=(6,) * ndim, sort_interval=1)
    sim = pic.Pic(cfg)
    sim.load_particles(x, u, np.full(n, -0.37), rqm=-1.0)
    print("units", ndim, order, move, "chunk", sim.info().chunk, flush=True)
    sim.rho_snapshot()
    rho0 = sim.rho()
    sim.step(1)
    rate = np.abs(sim.rho() - rho0).max() / dt
    assert rate > 0
    assert np.abs(sim.charge_residual()).max() <= 1e-4 * rate
    sim.close()
