"""Resident steps of two-word addresses against the step kernels, bit for bit.
A solver or a batch of addresses of at most 62 bits keeps one word; beside a
partner of more than 62 bits a batch keeps two.  Also the buckets that may
hold more addresses than the hash of a workgroup (4096 slots a bucket, 2048 in
the two-word hash): the launch that is not begun, the launch that ends, and
steps in between."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SHAPE = dict(lds_slots=2048, block=512, spawn_block=256)
RING = dict(model=0, M=8, N=8, u=4.0, dtau=1e-3, target_walkers=2e3, seed=11, table_capacity=8192,
            spawn_capacity=40000, addr_words=2, **SHAPE)
MOM = dict(RING, model=1, u=2.0, dtau=5e-4)
LATTICE = dict(RING, model=2, M=12, N=12, lx=4, t=0.1, u=1.0, g=0.5, dtau=5e-3)
CASES = {
    "ring, one bucket": (dict(RING, buckets=1), (1, 2, 250, 400)),
    "ring, 64 buckets": (dict(RING, buckets=64), (250, 250)),
    "ring, early": (dict(RING, buckets=4, flags=32), (250, 250)),
    "ring, initiator, early": (dict(RING, buckets=4, initiator=2.0, flags=32), (250, 250)),
    "ring, every column exact": (dict(RING, buckets=4, t_rel=0.0, spawn_capacity=200000), (250, 250)),
    "ring, 8192 buckets": (dict(RING, buckets=8192, table_capacity=16384, spawn_capacity=160000), (150, 150)),
    "ring, 16384 buckets: not resident": (dict(RING, buckets=16384, table_capacity=32768, spawn_capacity=320000), (60,)),
    "momentum": (dict(MOM, M=9, N=9, buckets=8, spawn_capacity=80000), (1, 300)),
    "momentum, initiator, few addresses": (dict(MOM, M=7, N=7, target_walkers=2e4, buckets=4, initiator=3.0,
                                                table_capacity=4000, spawn_capacity=160000), (300, 300)),
    "lattice": (dict(LATTICE, buckets=16), (300,)),
    "several passes": (dict(RING, M=11, N=11, target_walkers=6e4, buckets=64, table_capacity=200000,
                            spawn_capacity=400000), (300, 200)),
    "growth over several launches": (dict(RING, M=12, N=12, target_walkers=1e5, buckets=256, table_capacity=300000,
                                          spawn_capacity=600000), (400, 200)),
}


def _state(solver):
    a, v, shift, step = solver.get_state()
    o = np.lexsort(a.T)
    return a[o], v[o], shift, step


def _start(solver, spec, walkers=10.0):
    import paper_2601_19505_amd as fq
    a = fq.start_address(spec["model"], spec["M"], spec["N"], 2)
    solver.set_state([a], [walkers], 0.0, 0, ref=a, yref=10.0)


def _same(x, y):
    return np.array_equal(x[0], y[0]) and np.array_equal(x[1], y[1]) and x[2:] == y[2:]


def _partner(spec):
    wide = dict(spec, M=33, N=33, u=0.1, t=1.0, dtau=1e-4, target_walkers=100.0, seed=5, buckets=1, table_capacity=4096,
                spawn_capacity=20000, t_rel=1.0)
    if spec["model"] == 1:
        wide.update(M=32, N=32)
    if spec["model"] == 2:
        wide.update(M=36, N=36, lx=6, t=0.1, u=1.0)
    return wide


@pytest.mark.parametrize("name", list(CASES))
def test_two_words(name):
    import paper_2601_19505_amd as fq
    spec, calls = CASES[name]
    print("[words]", name, flush=True)
    batch, solo = fq.Batch([spec, _partner(spec)]), fq.Solver(**spec)
    solo.set_timing(True)
    _start(batch.instance(0), spec)
    _start(batch.instance(1), _partner(spec))
    _start(solo, spec)
    for n in calls:
        got, want = batch.run(n)[0], solo.run(n)
        for f in want.dtype.names:
            assert np.array_equal(got[f], want[f]), (n, f, int(np.argmax(got[f] != want[f])))
    assert _same(_state(batch.instance(0)), _state(solo))
    batch.close()
    solo.close()


@pytest.mark.parametrize("R, spec", [
    (2, dict(RING, M=32, N=32, u=0.1, target_walkers=5e2, buckets=8)),
    (3, dict(RING, M=32, N=32, u=0.1, target_walkers=2e3, buckets=16, table_capacity=60000, spawn_capacity=200000)),
    (2, dict(MOM, M=32, N=32, u=0.1, t=0.1, target_walkers=1e3, buckets=16, initiator=3.0, table_capacity=60000,
             spawn_capacity=200000)),
])
def test_two_word_replicas(R, spec):
    import paper_2601_19505_amd as fq
    print("[words] replicas", R, flush=True)
    specs = [dict(spec, seed=70 + i) for i in range(R)]
    a, b = fq.Batch(specs), fq.Batch(specs)
    for x in (a, b):
        for i in range(R):
            _start(x.instance(i), spec, 10.0 + i)
    b.instance(0).set_timing(True)
    for n in (100, 200):
        (ra, oa, ia), (rb, ob, ib) = a.run_replicas(n), b.run_replicas(n)
        assert ra.tobytes() == rb.tobytes() and oa.tobytes() == ob.tobytes() and ia == ib, n
    for i in range(R):
        assert _same(_state(a.instance(i)), _state(b.instance(i))), i
    a.close()
    b.close()


# 4096 slots a bucket, twice the two-word hash of a workgroup
LARGE = dict(RING, M=32, N=32, u=0.1, lds_slots=4096, block=512)


@pytest.mark.parametrize("name, more, calls", [
    # items to 1024 a bucket are stepped here, and more by the step kernels
    ("one bucket", dict(buckets=1, target_walkers=3e2, table_capacity=4000, spawn_capacity=20000), (100, 200)),
    ("launches that end", dict(buckets=4, target_walkers=6e3, table_capacity=16000, spawn_capacity=60000), (400, 200)),
    ("initiator", dict(buckets=16, target_walkers=4e3, initiator=3.0, table_capacity=30000, spawn_capacity=90000),
     (300, 200)),
])
def test_buckets_larger_than_the_hash(name, more, calls):
    import paper_2601_19505_amd as fq
    spec = dict(LARGE, **more)
    print("[words] large:", name, flush=True)
    a, b = fq.Solver(**spec), fq.Solver(**spec)
    b.set_timing(True)
    for s in (a, b):
        _start(s, spec)
    for n in calls:
        assert a.run(n).tobytes() == b.run(n).tobytes(), n
    assert _same(_state(a), _state(b))
    a.close()
    b.close()


def _of_one_bucket(spec, most, n):
    """n addresses that share one of the 8 buckets of `spec`: a state comes
    back bucket after bucket, so an entry's neighbours are of its bucket."""
    import paper_2601_19505_amd as fq
    import synthetic
    occ = synthetic.random_occupations(np.random.default_rng(7), spec["M"], spec["N"], most)
    a = fq.encode_many(occ, 2)
    one = fq.Solver(**spec)
    one.set_state(a, np.ones(len(a)), 0.0, 0, ref=a[0])
    a, _, _, _ = one.get_state()
    one.close()
    return a[:n]


@pytest.mark.parametrize("n, value, shift, calls", [
    (2200, 0.3, 0.0, (2, 100)),    # more than the hash of a workgroup: not begun
    (1760, 1.0, 100.0, (20, 20)),  # begun; the second step has two attempts an entry, and then it is more
])
def test_a_bucket_that_fills_the_hash(n, value, shift, calls):
    """All addresses in one bucket of 8: fewer items than the limit of a
    launch, and more in that bucket than its hash has slots."""
    import paper_2601_19505_amd as fq
    spec = dict(LARGE, M=33, N=31, buckets=8, table_capacity=30000, spawn_capacity=60000, target_walkers=2e3)
    print("[words] one bucket", n, flush=True)
    a = _of_one_bucket(spec, 24000, n)
    v = np.full(len(a), value)
    x, y = fq.Solver(**spec), fq.Solver(**spec)
    y.set_timing(True)
    for s in (x, y):
        s.set_state(a, v, shift, 0, ref=a[0])
    for k in calls:
        assert x.run(k).tobytes() == y.run(k).tobytes(), k
    assert y.debug_counters()["max_load"] > 2048
    assert _same(_state(x), _state(y))
    x.close()
    y.close()
