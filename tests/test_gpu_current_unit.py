"""The fixed point of a work item's current tile (two-phase kernels) where its
bounds could fail: particles whose momentum is not a number in FP32."""
import numpy as np
import pytest

from parity import J_TOL, rel_max

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx", [(48, 40), (16, 12, 16), (32, 16, 16)], ids=lambda n: "x".join(map(str, n)))
@pytest.mark.parametrize("order", [1, 2, 3])
def test_an_infinite_momentum_does_not_take_its_neighbours_current(nx, order):
    """1e39 is finite in FP64 and infinite in FP32: the particle adds nothing to
    the current, and the others' current stays what it is without it."""
    from paper_1503_00276_amd import pic

    rng = np.random.default_rng(order)
    ppc = 2
    n = ppc * int(np.prod(nx))
    x = rng.random((n, len(nx))) * np.asarray(nx) * 0.2
    u, w = rng.normal(0, 0.3, (n, 3)), np.full(n, -1.0 / ppc)
    got = []
    for extra in (0, 1):
        sim = pic.Pic(pic.Config(ndim=len(nx), nx=nx, dx=(0.2,) * len(nx), dt=0.08, shape_order=order))
        ux = np.concatenate([u, np.full((extra, 3), [[1e39, 0.0, 1.0]])])
        print("infinite", nx, order, extra, flush=True)
        sim.load_particles(np.concatenate([x, x[:extra]]), ux, np.concatenate([w, w[:extra]]), rqm=-1.0)
        sim.step(1)
        got.append(sim.current())
        sim.close()
    assert rel_max(got[1], got[0]) <= J_TOL
