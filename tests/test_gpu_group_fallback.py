"""Instances of a batch that outgrow their resident workgroups in the middle of
a chunk, at different steps, beside one that does not: the step kernels make
what is left of the chunk for all of them together, and every instance has the
rows and the state it has alone."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# buckets of 4096 slots, twice the two-word hash: resident to 1024 items a bucket
SPEC = dict(model=0, M=32, N=32, u=0.1, dtau=1e-3, addr_words=2, lds_slots=4096, block=512, spawn_block=256, buckets=4,
            table_capacity=16000, spawn_capacity=60000)


def _state(solver):
    a, v, shift, step = solver.get_state()
    o = np.lexsort(a.T)
    return a[o], v[o], shift, step


def test_instances_that_outgrow_their_workgroups():
    import paper_2601_19505_amd as fq
    a = fq.start_address(0, SPEC["M"], SPEC["N"], 2)
    # walkers at the start, target
    runs = [(10.0, 3e3), (300.0, 3.5e3), (10.0, 2e2), (1500.0, 4e3)]
    specs = [dict(SPEC, target_walkers=t, seed=50 + i) for i, (_, t) in enumerate(runs)]
    batch, solo = fq.Batch(specs), [fq.Solver(**sp) for sp in specs]
    for i, (w, _) in enumerate(runs):
        for s in (batch.instance(i), solo[i]):
            s.set_state([a], [w], 0.0, 0, ref=a, yref=10.0)
        solo[i].set_timing(True)
    # the second call goes over the end of a chunk of 4096 steps
    for n in (350, 4200, 30):
        print("[fallback]", n, flush=True)
        rows = batch.run(n)
        for i, s in enumerate(solo):
            assert rows[i].tobytes() == s.run(n).tobytes(), (n, i)
    for i, s in enumerate(solo):
        x, y = _state(batch.instance(i)), _state(s)
        assert np.array_equal(x[0], y[0]) and np.array_equal(x[1], y[1]) and x[2:] == y[2:], i
        s.close()
    batch.close()


def test_many_of_them_share_their_launches():
    """Sixteen equal instances take little longer than one, and not sixteen times."""
    import time

    import paper_2601_19505_amd as fq
    a = fq.start_address(0, SPEC["M"], SPEC["N"], 2)
    took = {}
    for n in (1, 16):
        batch = fq.Batch([dict(SPEC, target_walkers=4e3, seed=50 + i) for i in range(n)])
        for i in range(n):
            batch.instance(i).set_state([a], [1500.0], 0.0, 0, ref=a, yref=10.0)
        t = time.perf_counter()
        rows = batch.run(1000)
        took[n] = time.perf_counter() - t
        assert np.all(rows["len"][:, -1] + rows["spawns"][:, -1] > 4 * 1024)
        batch.close()
    print("[fallback]", took, flush=True)
    assert took[16] < 5 * took[1]
