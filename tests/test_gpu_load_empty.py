"""Loading into a store whose particles are all gone (the r-z wall took them): its
counters of checks and rebins go on."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_an_emptied_store_keeps_its_counters():
    from paper_1503_00276_amd import pic

    nz, nr, d = 16, 12, 0.2
    sim = pic.Pic(pic.Config(ndim=2, nx=(nz, nr), dx=(d, d), dt=0.1, shape_order=1, geometry=pic.PIC_GEOM_RZ,
                             capacity=1000))
    rng = np.random.default_rng(2)
    n = 200
    x = np.stack([rng.random(n) * nz * d, np.full(n, (nr - 1) * d)], 1)
    u = np.tile((0.0, 5.0, 0.0), (n, 1))
    print("emptied store", flush=True)
    sim.load_particles(x, u, np.full(n, -1e-6), rqm=-1.0)
    sim.step(6)
    sim.sync()
    _, left, sorts, checks = sim.counts()
    assert left == 0 and sorts >= 1 and checks == 6
    sim.load_particles(x[:50], u[:50] * 0.0, np.full(50, -1e-6), rqm=-1.0)
    assert list(sim.counts()[1:]) == [50, sorts, checks]
    xs, us, ws = sim.state()
    assert len(ws) == 50 and np.all(us == 0.0)
    sim.step(2)
    sim.sync()
    assert sim.counts()[1] == 50 and sim.counts()[3] == checks + 2
    sim.close()
