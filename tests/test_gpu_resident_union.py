"""Two runs for excited states that grow until the addresses of both outgrow
the hash of a resident workgroup, while the second run's own still fit it: the
step is made by the step kernels, whose hash is twice the bucket's, and rows
and states equal theirs bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# one workgroup a run and two buckets: its hash of 4096 slots meets what the
# step kernels keep in two hashes of 8192
SPEC = dict(model=0, M=10, N=10, u=4.0, dtau=1e-3, table_capacity=16384, spawn_capacity=60000, buckets=2,
            lds_slots=4096, block=512, spawn_block=256)


def _batch(specs, step_kernels):
    import paper_2601_19505_amd as fq
    batch = fq.Batch(specs)
    for i, sp in enumerate(specs):
        W = sp.get("addr_words", 1)
        ref = fq.start_address(sp["model"], sp["M"], sp["N"], W)
        occ = [1] * sp["M"]
        if i:
            occ[0], occ[1] = 2, 0
        batch.instance(i).set_state([fq.encode(occ, W)], [10.0 + 3 * i], 0.0, 0, ref=ref, yref=10.0)
    if step_kernels:
        batch.instance(0).set_timing(True)
    return batch


def _state(solver):
    a, v, shift, step = solver.get_state()
    o = np.lexsort(a.T)
    return a[o], v[o], shift, step


@pytest.mark.parametrize("seed", [60, 62, 64])
@pytest.mark.parametrize("target", [2e3, 3e3, 4e3])
def test_growth_past_the_hash_of_both_runs(target, seed):
    print("[union]", target, seed, flush=True)
    specs = [dict(SPEC, target_walkers=target, seed=seed + i) for i in range(2)]
    a, b = _batch(specs, False), _batch(specs, True)
    for n in (330, 40):
        (ra, ia), (rb, ib) = a.run_spectral(n), b.run_spectral(n)
        assert ra.tobytes() == rb.tobytes() and ia == ib, n
    for i in range(2):
        x, y = _state(a.instance(i)), _state(b.instance(i))
        assert np.array_equal(x[0], y[0]) and np.array_equal(x[1], y[1]) and x[2:] == y[2:], i
    # the addresses of the second run alone came to more than the hash holds
    assert b.instance(1).debug_counters()["max_load"] > 2100
    a.close()
    b.close()
