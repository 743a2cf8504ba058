"""The item counts of a launch that holds many stores: a store per lane, 64 at
a time, with an exclusive sum over them.  Batches of one store, of a few, of
one more and one less than 64 and of more than two chunks, with particle
counts that differ from instance to instance; each instance must be to the bit
what it is when it runs alone (int64 sums, so the order of items is free)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count", [1, 3, 63, 64, 65, 131])
def test_instances_of_a_group_run_as_alone(count):
    from paper_1503_00276_amd import pic

    cfg = pic.Config(ndim=2, nx=(16, 12), dx=(0.2, 0.2), dt=0.1, shape_order=1, tile=(8, 6), sort_interval=2,
                     accumulator=pic.PIC_ACC_FIXED64)
    rng = np.random.default_rng(count)
    data = []
    for i in range(count):
        n = 1 if i % 7 == 3 else int(rng.integers(20, 900))
        x = rng.random((n, 2)) * np.array([16, 12]) * 0.2 * 0.999
        data.append((x, rng.normal(size=(n, 3)) * 0.4, np.full(n, -0.01 * (1 + i % 5))))
    batch = pic.PicBatch([cfg] * count)
    for i, (x, u, w) in enumerate(data):
        batch.load_particles(i, x, u, w)
    print("batch groups", count, flush=True)
    batch.step(7)
    for i in sorted({0, 1 % count, count // 2, min(63, count - 1), min(64, count - 1), count - 1}):
        alone = pic.Pic(cfg)
        alone.load_particles(*data[i])
        alone.step(7)
        for a, b in zip(batch.fields(i), alone.fields()):
            assert np.array_equal(a, b)
        assert np.array_equal(batch.current(i), alone.current())
        alone.close()
    batch.close()
