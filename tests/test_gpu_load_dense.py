"""Loading cells of very different particle numbers: no particle of a tile is
lost, doubled or misplaced where the ranks of its cells are interleaved (equal
counts, counts that differ by one, empty cells, one cell that holds all, tiles
larger than a workgroup, ragged ones)."""
import numpy as np
import pytest

from test_gpu_load import _check

pytestmark = pytest.mark.gpu

DX, XMIN = (0.2, 0.25, 0.22), (0.0, 0.0, 0.0)


def _counts(kind, ncell, rng):
    if kind == "equal":
        return np.full(ncell, 7)
    if kind == "one apart":
        return 600 + np.arange(ncell) % 3
    if kind == "all different":
        return rng.permutation(ncell)
    if kind == "one cell":
        c = np.zeros(ncell, int)
        c[ncell // 2] = 20000
        return c
    c = rng.choice([0, 0, 1, 2, 511, 512, 513, 1500], ncell)  # "mixed"
    return c


@pytest.mark.parametrize("kind", ["equal", "one apart", "all different", "one cell", "mixed"])
@pytest.mark.parametrize("nx,tile", [((16, 16), (8, 8)), ((19, 20), (16, 20)), ((8, 11, 7), (4, 4, 7))],
                         ids=["8x8", "16x20", "4x4x7"])
def test_every_particle_is_stored_once(nx, tile, kind):
    from paper_1503_00276_amd import pic

    dim = len(nx)
    rng = np.random.default_rng(len(kind))
    c = np.repeat(np.indices(nx).reshape(dim, -1).T, _counts(kind, int(np.prod(nx)), rng), 0)
    n = len(c)
    part = ((c + rng.random((n, dim))) * np.asarray(DX[:dim]), rng.normal(0, 0.2, (n, 3)), rng.uniform(-1, -0.1, n))
    order = rng.permutation(n)
    part = tuple(a[order] for a in part)
    cfg = pic.Config(ndim=dim, nx=nx, dx=DX[:dim], dt=0.05, shape_order=1, tile=tile, sort_interval=1,
                     accumulator=pic.PIC_ACC_FIXED64)
    sim = pic.Pic(cfg)
    print("dense", nx, kind, n, flush=True)
    sim.load_particles(*part, rqm=-1.0)
    _check(sim, [part], nx, DX, XMIN)
    sim.step(2)
    assert sim.counts()[1] == n
    sim.close()
