"""The rebin check of a moving window on both sides of the largest store that the
field step plans (16,384 tiles): with the int64 current the tiling changes no
arithmetic, so after several shifts, with particles removed at the back and
injected at the front (cold and thermal), the whole state equals, bit for bit,
that of the same box in a few large tiles."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,tile,ref", [((387, 384), (3, 3), (43, 32)), ((384, 384), (3, 3), (32, 32)),
                                         ((99, 96), (3, 3), (33, 32))],
                         ids=["16512_tiles", "16384_tiles", "1056_tiles"])
@pytest.mark.parametrize("uth", [0.0, 0.2])
def test_window_in_many_tiles(nx, tile, ref, uth):
    from paper_1503_00276_amd import pic

    rng = np.random.default_rng(4)
    n = 2 * nx[0] * nx[1]
    x = rng.random((n, 2)) * np.asarray(nx) * 0.2
    u, w = rng.normal(0, 0.8, (n, 3)), np.full(n, -0.5)
    got = []
    for t in (tile, ref):
        sim = pic.Pic(pic.Config(ndim=2, nx=nx, dx=(0.2, 0.2), dt=0.1, shape_order=1, tile=t, ion_density=1.0,
                                 accumulator=pic.PIC_ACC_FIXED64, move_window=1, inject_ppc=(2, 1, 1), inject_w=-0.5,
                                 inject_uth=uth, inject_seed=5))
        print("window tiles", nx, t, uth, flush=True)
        sim.load_particles(x, u, w, rqm=-1.0)
        sim.step(9)  # four shifts
        sim.sync()
        got.append((*sim.state(), *sim.fields(), sim.current()))
        assert sim.counts()[2] >= 4
        sim.close()
    for p, q in zip(*got):
        np.testing.assert_array_equal(p, q)
