"""The default chunk follows the particles of a store, however they are loaded: at
once, in slices that grow the store, or in slices within its capacity; a chunk
that was asked for stays."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

NX, PPC = (192, 160), 12


def _plasma():
    rng = np.random.default_rng(3)
    n = PPC * NX[0] * NX[1]
    x = rng.random((n, 2)) * np.asarray(NX) * 0.2
    return x, rng.normal(0, 0.2, (n, 3)), np.full(n, -1.0 / PPC)


@pytest.mark.parametrize("kind", ["two-phase", "int64", "r-z"])
def test_chunk_of_a_store_loaded_in_slices(kind):
    from paper_1503_00276_amd import pic

    kw = {"two-phase": {}, "int64": {"accumulator": pic.PIC_ACC_FIXED64},
          "r-z": {"geometry": pic.PIC_GEOM_RZ}}[kind]
    part = _plasma()
    n = len(part[2])
    got = {}
    for how, extra in (("at once", {}), ("growing", {}), ("within the capacity", {"capacity": n}),
                       ("asked", {"chunk": 320, "capacity": n})):
        sim = pic.Pic(pic.Config(ndim=2, nx=NX, dx=(0.2, 0.2), dt=0.1, shape_order=1, **kw, **extra))
        first = None
        print("chunk", kind, how, flush=True)
        for i in np.array_split(np.arange(n), 1 if how == "at once" else 8):
            keep = i[part[0][i, 1] < (NX[1] - 1) * 0.2]  # (off the wall)
            sim.load_particles(*(a[keep] for a in part), rqm=-1.0)
            first = first or sim.info().chunk
        got[how] = sim.info().chunk
        assert how == "at once" or first <= got[how]
        sim.step(3)
        sim.sync()
        sim.close()
    assert got["at once"] > 256 and got["asked"] == 320
    assert got["growing"] == got["at once"] and got["within the capacity"] == got["at once"]
