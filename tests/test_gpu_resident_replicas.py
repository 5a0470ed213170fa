"""Replicas stepped together by resident workgroups against the step and
overlap kernels, which a batch uses while an instance's kernels are timed:
rows, overlaps and final states bit for bit, over replica, bucket and
workgroup counts, address widths, sizes that outgrow the workgroups, and a
replica that ends with an error."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

BASE = dict(model=0, M=8, N=8, u=4.0, dtau=1e-3, target_walkers=2e3, table_capacity=8192, spawn_capacity=40000)
MOM = dict(BASE, model=1, u=2.0, dtau=5e-4)


def _batch(specs, walkers, step_kernels):
    import paper_2601_19505_amd as fq
    batch = fq.Batch(specs)
    for i, sp in enumerate(specs):
        a = fq.start_address(sp["model"], sp["M"], sp["N"], sp.get("addr_words", 1))
        batch.instance(i).set_state([a], [walkers[i]], 0.0, 0, ref=a, yref=10.0)
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
    (2, dict(BASE, buckets=1), (50, 200)),                        # no workgroup pair: step kernels
    (2, dict(BASE, buckets=2), (1, 2, 3, 300)),
    (2, dict(BASE, buckets=64), (400,)),
    (3, dict(BASE, buckets=8), (7, 300)),
    (3, dict(BASE, buckets=4, addr_words=2), (200, 200)),
    (8, dict(BASE, buckets=64, target_walkers=5e2), (250,)),
    (2, dict(BASE, buckets=8192, table_capacity=16384, spawn_capacity=160000), (120,)),
    (4, dict(BASE, buckets=8192, table_capacity=16384, spawn_capacity=160000), (60,)),   # 512 workgroups: step kernels
    (2, dict(MOM, buckets=8), (1, 300)),
    (2, dict(MOM, M=18, N=18, u=1.0, buckets=32, table_capacity=40000, spawn_capacity=200000), (250,)),
    (2, dict(MOM, M=7, N=7, buckets=8, addr_words=2, initiator=3.0), (300,)),
    (2, dict(BASE, model=2, M=9, N=9, lx=3, t=0.1, u=1.0, g=1.0, dtau=5e-3, buckets=4), (300,)),
    (2, dict(BASE, buckets=4, flags=32), (200,)),                 # early compression: step kernels
    (2, dict(BASE, M=9, N=9, target_walkers=4e3, buckets=2, lds_slots=4096), (500, 200)),  # outgrows two workgroups
    # few addresses and many records; more addresses than the hashes hold
    (2, dict(MOM, M=7, N=7, target_walkers=3e4, buckets=4, table_capacity=6000, spawn_capacity=200000), (300, 100)),
    (2, dict(BASE, M=11, N=11, target_walkers=3e4, buckets=16, table_capacity=60000, spawn_capacity=200000), (400, 100, 50)),
    (2, dict(BASE, M=12, N=12, target_walkers=4e4, buckets=256, lds_slots=2048, block=512, table_capacity=200000,
             spawn_capacity=400000), (500, 300)),
])
def test_resident_replicas_equal_the_step_kernels(R, spec, calls):
    print("[replicas]", R, spec, flush=True)
    specs = [dict(spec, seed=70 + i) for i in range(R)]
    walkers = [10.0 + i for i in range(R)]
    a, b = _batch(specs, walkers, False), _batch(specs, walkers, True)
    for n in calls:
        ra, oa, ia = a.run_replicas(n)
        rb, ob, ib = b.run_replicas(n)
        assert ra.tobytes() == rb.tobytes() and oa.tobytes() == ob.tobytes() and ia == ib, n
        assert np.all(oa[-1] != 0.0)
    _same_states(a, b, R)
    a.close()
    b.close()


@pytest.mark.parametrize("bad", [0, 1, 2])
@pytest.mark.parametrize("kind", ["capacity", "diverged"])
def test_a_replica_that_fails_ends_the_others_where_the_step_kernels_do(kind, bad):
    import paper_2601_19505_amd as fq
    spec = dict(BASE, buckets=8, table_capacity=4000, spawn_capacity=16000)
    specs = [dict(spec, seed=80 + i, target_walkers=3e2) for i in range(3)]
    walkers = [10.0] * 3
    if kind == "capacity":
        specs[bad]["target_walkers"] = 1e5
    else:
        # every column exact, so that few addresses carry 2^44 walkers within a few steps
        specs = [dict(s, t_rel=0.0, table_capacity=8000, spawn_capacity=200000) for s in specs]
        walkers[bad] = 1.7e13
        specs[bad]["target_walkers"] = 1e14
    got = []
    for kernels in (False, True):
        batch = _batch(specs, walkers, kernels)
        with pytest.raises(fq.FqError) as e:
            batch.run_replicas(400)
        rows = e.value.stats
        done = [int(np.count_nonzero(rows[i]["step"])) for i in range(3)]
        least = min(done)
        got.append((e.value.status, e.value.instance, done, rows.tobytes(), e.value.overlaps[:least].tobytes(),
                    [_state(batch.instance(i)) for i in range(3)]))
        batch.close()
    x, y = got
    print("[replicas]", kind, bad, x[:3], flush=True)
    assert x[:3] == y[:3] and x[1] == bad and x[2][bad] < 400
    assert x[3] == y[3] and x[4] == y[4]
    for p, q in zip(x[5], y[5]):
        assert np.array_equal(p[0], q[0]) and np.array_equal(p[1], q[1]) and p[2:] == q[2:]
