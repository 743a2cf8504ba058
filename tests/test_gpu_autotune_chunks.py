"""The autotuner where the stores' default chunks differ (they follow the particles
loaded): a search that leaves the chunk out keeps every store's own, and the
layout it starts from is the one in force."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _pic():
    from paper_1503_00276_amd import pic

    return pic


def _plasma(nx, ppc, seed):
    rng = np.random.default_rng(seed)
    n = ppc * int(np.prod(nx))
    x = rng.random((n, len(nx))) * np.asarray(nx) * 0.2
    return x, rng.normal(0, 0.1, (n, 3)), np.full(n, -1.0 / ppc)


def _cfg(pic, nx):
    return pic.Config(ndim=2, nx=nx, dx=(0.2, 0.2), dt=0.1, shape_order=1, ion_density=1.0)


@pytest.mark.parametrize("what", ["tile", "sort"])
def test_uneven_boxes_of_a_batch_keep_their_chunks(what):
    pic = _pic()
    boxes = [((48, 48), 8), ((256, 192), 12)]
    batch = pic.PicBatch([_cfg(pic, nx) for nx, _ in boxes])
    for k, (nx, ppc) in enumerate(boxes):
        batch.load_particles(k, *_plasma(nx, ppc, k), rqm=-1.0)
    batch.step(2)
    chunks = [batch.info(k).chunk for k in range(2)]
    assert chunks[0] != chunks[1]
    print("batch chunks", what, chunks, flush=True)
    res = batch.autotune(trial_steps=2, what={"tile": pic.PIC_TUNE_TILE, "sort": pic.PIC_TUNE_SORT}[what])
    assert [batch.info(k).chunk for k in range(2)] == chunks
    assert res["chunk"] == chunks[0]
    batch.step(3)
    batch.close()


def test_a_small_species_does_not_set_the_chunk_of_a_large_one():
    pic = _pic()
    sim = pic.Pic(_cfg(pic, (256, 192)))
    small = tuple(a[:2000] for a in _plasma((256, 192), 1, 5))
    large = _plasma((256, 192), 12, 6)
    sim.load_particles(*small, rqm=-1.0, species=0)
    small_chunk = sim.info().chunk
    sim.load_particles(*large, rqm=-1.0, species=1)
    chunk = sim.info().chunk  # (that of the last species in use)
    assert chunk > small_chunk
    sim.step(2)
    sim.autotune(trial_steps=2, what=pic.PIC_TUNE_SORT)
    assert sim.info().chunk == chunk
    # a search of the chunk gives all stores the one it finds
    res = sim.autotune(trial_steps=2, what=pic.PIC_TUNE_CHUNK)
    assert res["chunk"] in (small_chunk, 512, 1024, 2048)
    sim.step(2)
    sim.close()
