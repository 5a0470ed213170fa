"""Two runs for excited states stepped together by resident workgroups against
the step and projection kernels, which a batch uses while an instance's
kernels are timed: rows and final states bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

BASE = dict(model=0, M=8, N=8, u=4.0, dtau=1e-3, target_walkers=2e3, table_capacity=16384, spawn_capacity=60000,
            lds_slots=2048, block=512, spawn_block=256)


def _batch(specs, walkers, step_kernels):
    import paper_2601_19505_amd as fq
    batch = fq.Batch(specs)
    for i, sp in enumerate(specs):
        W = sp.get("addr_words", 1)
        a = fq.start_address(sp["model"], sp["M"], sp["N"], W)
        occ = [1] * sp["M"]
        if i:
            occ[0], occ[i] = 2, 0
        b = fq.encode(occ, W) if sp["N"] == sp["M"] and sp["model"] != 1 else a
        batch.instance(i).set_state([b], [walkers[i]], 0.0, 0, ref=a, yref=10.0)
    if step_kernels:
        batch.instance(0).set_timing(True)
    return batch


def _state(solver):
    a, v, shift, step = solver.get_state()
    o = np.lexsort(a.T)
    return a[o], v[o], shift, step


def _same_states(a, b, n):
    for i in range(n):
        x, y = _state(a.instance(i)), _state(b.instance(i))
        assert np.array_equal(x[0], y[0]) and np.array_equal(x[1], y[1]) and x[2:] == y[2:], i


@pytest.mark.parametrize("R, spec, calls", [
    (2, dict(BASE, buckets=1), (100,)),                           # step kernels
    (2, dict(BASE, buckets=2), (1, 2, 3, 300)),
    (2, dict(BASE, buckets=8, target_walkers=5e3), (300, 100)),
    (2, dict(BASE, buckets=64), (400,)),
    (3, dict(BASE, buckets=8), (100,)),                           # three runs: step kernels
    (2, dict(BASE, buckets=8192, table_capacity=32768, spawn_capacity=200000), (100,)),
    (2, dict(BASE, M=32, N=32, u=0.1, target_walkers=5e2, addr_words=2, buckets=8), (300,)),   # 63 bits
    (2, dict(BASE, buckets=8, initiator=2.0), (300,)),
    (2, dict(BASE, buckets=4, flags=32), (100,)),                 # early compression: step kernels
    (2, dict(BASE, model=2, M=9, N=9, lx=3, t=0.1, u=1.0, g=1.0, dtau=5e-3, buckets=4), (300,)),
    (2, dict(BASE, model=1, u=2.0, dtau=5e-4, buckets=8), (200,)),   # equal runs: the second vanishes or not alike
    (2, dict(BASE, M=9, N=9, target_walkers=5e3, buckets=8), (500, 100)),   # outgrows four workgroups a run
    # few addresses and many records; more addresses than the hashes hold
    (2, dict(BASE, M=6, N=6, target_walkers=3e4, buckets=2, table_capacity=3000, spawn_capacity=200000), (400, 100)),
    (2, dict(BASE, M=10, N=10, target_walkers=2e4, buckets=32, table_capacity=60000, spawn_capacity=200000), (400, 100)),
    (2, dict(BASE, M=12, N=12, target_walkers=3e4, buckets=256, table_capacity=200000, spawn_capacity=400000),
     (400, 200)),
])
def test_resident_runs_equal_the_step_kernels(R, spec, calls):
    print("[spectral]", R, spec, flush=True)
    specs = [dict(spec, seed=60 + i) for i in range(R)]
    walkers = [10.0 + 3 * i for i in range(R)]
    a, b = _batch(specs, walkers, False), _batch(specs, walkers, True)
    for n in calls:
        ra, ia = a.run_spectral(n)
        rb, ib = b.run_spectral(n)
        assert ra.tobytes() == rb.tobytes() and ia == ib, n
    _same_states(a, b, R)
    a.close()
    b.close()


@pytest.mark.parametrize("bad", [0, 1])
@pytest.mark.parametrize("kind", ["table", "slab", "diverged"])
def test_a_run_that_fails_ends_where_the_step_kernels_do(kind, bad):
    import paper_2601_19505_amd as fq
    spec = dict(BASE, buckets=8, table_capacity=3000, spawn_capacity=20000)
    if kind == "slab":
        spec.update(table_capacity=8000, spawn_capacity=8000)
    specs = [dict(spec, seed=80 + i, target_walkers=3e2) for i in range(2)]
    walkers = [10.0] * 2
    if kind == "diverged":
        specs = [dict(s, t_rel=0.0, table_capacity=8000, spawn_capacity=200000) for s in specs]
        walkers[bad] = 1.7e13
        specs[bad]["target_walkers"] = 1e14
    else:
        specs[bad]["target_walkers"] = 1e5
    got = []
    for kernels in (False, True):
        batch = _batch(specs, walkers, kernels)
        with pytest.raises(fq.FqError) as e:
            batch.run_spectral(400)
        rows = e.value.stats
        done = [int(np.count_nonzero(rows[i]["step"])) for i in range(2)]
        got.append((e.value.status, e.value.instance, done, rows.tobytes(), [_state(batch.instance(i)) for i in range(2)]))
        batch.close()
    x, y = got
    print("[spectral]", kind, bad, x[:3], y[:3], flush=True)
    assert x[:3] == y[:3] and x[2][x[1]] < 400
    assert x[3] == y[3]
    for p, q in zip(x[4], y[4]):
        assert np.array_equal(p[0], q[0]) and np.array_equal(p[1], q[1]) and p[2:] == q[2:]
