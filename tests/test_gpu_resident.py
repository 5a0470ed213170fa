"""Resident steps (one launch for many steps of a small instance) against the
step kernels, which a solver uses while its kernels are timed: every row and
the final state bit for bit, over bucket counts, workgroup counts, models,
address widths, options and sizes at which the resident path splits a batch,
outgrows its workgroups or ends with an error."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _fq():
    import paper_2601_19505_amd as fq
    return fq


def _state(solver):
    a, v, shift, step = solver.get_state()
    o = np.lexsort(a.T)
    return a[o], v[o], shift, step


def _start(solver, spec, walkers):
    fq = _fq()
    a = fq.start_address(spec["model"], spec["M"], spec["N"], spec.get("addr_words", 1))
    solver.set_state([a], [walkers], 0.0, 0, ref=a, yref=10.0)


def _pair(spec, walkers=10.0):
    """A solver that may take resident steps and one that may not."""
    fq = _fq()
    out = []
    for timed in (False, True):
        s = fq.Solver(**spec)
        if timed:
            s.set_timing(True)
        _start(s, spec, walkers)
        out.append(s)
    return out


def _same(a, b, calls):
    for n in calls:
        ra, rb = a.run(n), b.run(n)
        for f in ra.dtype.names:
            assert np.array_equal(ra[f], rb[f]), (n, f, int(np.argmax(ra[f] != rb[f])))
    sa, sb = _state(a), _state(b)
    assert np.array_equal(sa[0], sb[0]) and np.array_equal(sa[1], sb[1]) and sa[2:] == sb[2:]


RING = dict(model=0, M=8, N=8, u=4.0, dtau=1e-3, target_walkers=2e3, seed=11, table_capacity=8192,
            spawn_capacity=40000)
CASES = {
    "ring, one bucket": dict(RING, buckets=1),
    "ring, two buckets": dict(RING, buckets=2),
    "ring, 64 buckets": dict(RING, buckets=64),
    "ring, 1024 buckets": dict(RING, buckets=1024),
    "ring, 2048 buckets: not resident": dict(RING, buckets=2048),
    "ring, two words": dict(RING, buckets=8, addr_words=2),
    "ring, 33 address bits": dict(RING, M=17, N=17, target_walkers=5e3, buckets=16, table_capacity=20000),
    "ring, early": dict(RING, buckets=4, flags=32),
    "ring, initiator": dict(RING, buckets=4, initiator=3.0),
    "ring, initiator, early, two words": dict(RING, buckets=4, initiator=2.0, flags=32, addr_words=2),
    "ring, every column exact": dict(RING, buckets=4, t_rel=0.0, spawn_capacity=200000),
    "ring, none exact, threshold": dict(RING, buckets=4, t_rel=np.inf, threshold=0.5, spawn_capacity=200000),
    "ring, two sites": dict(RING, M=2, N=9, target_walkers=500.0, buckets=2),
    "momentum": dict(RING, model=1, M=9, N=9, u=2.0, dtau=5e-4, buckets=8, spawn_capacity=80000),
    "momentum, early": dict(RING, model=1, M=8, N=8, u=2.0, dtau=5e-4, buckets=8, flags=32),
    "momentum, 35 bits, initiator": dict(RING, model=1, M=18, N=18, u=1.0, dtau=5e-4, buckets=32, initiator=3.0,
                                         table_capacity=40000, spawn_capacity=200000),
    "momentum, two words": dict(RING, model=1, M=7, N=7, u=2.0, dtau=5e-4, buckets=8, addr_words=2),
    "lattice, importance sampled": dict(RING, model=2, M=9, N=9, lx=3, t=0.1, u=1.0, g=1.0, dtau=5e-3, buckets=4),
    "lattice, two words": dict(RING, model=2, M=12, N=12, lx=4, t=0.1, u=1.0, g=0.5, dtau=5e-3, buckets=16,
                               addr_words=2),
    "one bucket in several batches": dict(RING, M=9, N=9, target_walkers=4e3, buckets=2),
    "growth over several launches": dict(RING, M=12, N=12, target_walkers=1e5, buckets=256, lds_slots=2048, block=512,
                                         table_capacity=300000, spawn_capacity=600000),
}


# the widest counters and beyond them; more records than hash slots, with few
# and with many distinct addresses; buckets that may outgrow the hash of a
# workgroup; attempts in several reserving groups
WIDE = {
    "4096 buckets": dict(RING, buckets=4096, table_capacity=16384),
    "8192 buckets, early": dict(RING, buckets=8192, flags=32, table_capacity=16384, spawn_capacity=160000),
    "8192 buckets, two words": dict(RING, buckets=8192, addr_words=2, table_capacity=16384, spawn_capacity=160000),
    "16384 buckets: not resident": dict(RING, buckets=16384, table_capacity=32768, spawn_capacity=320000),
    "few addresses, many records": dict(RING, model=1, M=7, N=7, u=2.0, dtau=5e-4, target_walkers=2e4, buckets=2,
                                        table_capacity=4000, spawn_capacity=160000),
    "few addresses, many records, initiator, two words": dict(
        RING, model=1, M=7, N=7, u=2.0, dtau=5e-4, target_walkers=2e4, buckets=4, addr_words=2, initiator=3.0,
        table_capacity=4000, spawn_capacity=160000, lds_slots=2048, block=512),
    "many addresses, several batches": dict(RING, M=11, N=11, target_walkers=6e4, buckets=64, lds_slots=2048, block=512,
                                            table_capacity=200000, spawn_capacity=400000),
    "buckets beyond the hash": dict(RING, M=9, N=9, target_walkers=6e3, buckets=4, addr_words=2, table_capacity=16000),
}


@pytest.mark.parametrize("name", list(WIDE))
def test_wide_resident_steps_equal_the_step_kernels(name):
    spec = WIDE[name]
    print("[resident]", name, spec, flush=True)
    a, b = _pair(spec)
    _same(a, b, (1, 250, 600))
    a.close()
    b.close()


@pytest.mark.parametrize("n", [64, 65, 130])
def test_a_batch_of_more_instances_than_a_launch_takes(n):
    """256 buckets need four workgroups an instance: 64 instances a launch."""
    fq = _fq()
    specs = [dict(RING, M=7 + i % 2, N=7 + i % 2, target_walkers=5e2, buckets=256, seed=90 + i, lds_slots=1024,
                  block=256, spawn_block=256) for i in range(n)]
    batch = fq.Batch(specs)
    for i, sp in enumerate(specs):
        _start(batch.instance(i), sp, 10.0)
    rows = [batch.run(k) for k in (3, 120)]
    for i in (0, 1, 63, n - 2, n - 1):
        s = fq.Solver(**specs[i])
        s.set_timing(True)
        _start(s, specs[i], 10.0)
        for got, k in zip(rows, (3, 120)):
            assert got[i].tobytes() == s.run(k).tobytes(), (i, k)
        sa, sb = _state(batch.instance(i)), _state(s)
        assert np.array_equal(sa[0], sb[0]) and np.array_equal(sa[1], sb[1])
        s.close()
    batch.close()


@pytest.mark.parametrize("name", list(CASES))
def test_resident_steps_equal_the_step_kernels(name):
    spec = CASES[name]
    print("[resident]", name, spec, flush=True)
    a, b = _pair(spec)
    _same(a, b, (1, 2, 250, 400))
    a.close()
    b.close()


@pytest.mark.parametrize("kind", ["table", "spawn", "hash"])
def test_a_full_table_slab_or_hash_stops_where_the_step_kernels_stop(kind):
    """The error leaves both at a completed step with the same rows; one
    bucket, so that both stop at the same one."""
    fq = _fq()
    # with every column exact an entry has about ten spawns: the slab fills long before the table
    room = dict(table=dict(table_capacity=600, spawn_capacity=8000),
                spawn=dict(table_capacity=2000, spawn_capacity=2000, t_rel=0.0),
                hash=dict(table_capacity=4000, spawn_capacity=20000, lds_slots=1024, block=256))[kind]
    spec = dict(RING, M=9, N=9, target_walkers=3e3, buckets=1)
    spec.update(room)
    got = []
    for s in _pair(spec):
        with pytest.raises(fq.FqError) as e:
            s.run(900)
        assert e.value.status == -2
        rows = e.value.stats
        got.append((rows[: int(np.count_nonzero(rows["step"]))], _state(s)))
        s.close()
    (ra, sa), (rb, sb) = got
    assert 50 < len(ra) < 900 and ra.tobytes() == rb.tobytes()
    assert np.array_equal(sa[0], sb[0]) and np.array_equal(sa[1], sb[1]) and sa[2:] == sb[2:]


def test_a_batch_of_unequal_instances_equals_its_solvers():
    """Instances that end a launch at different steps, one of them outgrowing
    its workgroups, beside a fresh state set between two calls."""
    fq = _fq()
    shape = dict(lds_slots=1024, block=256, spawn_block=256)
    specs = [dict(RING, M=m, N=m, target_walkers=t, buckets=k, seed=40 + i, table_capacity=int(1.6 * t) + 4096,
                  spawn_capacity=int(4 * t) + 20000, **shape)
             for i, (m, t, k) in enumerate([(6, 5e2, 1), (8, 2e3, 8), (10, 2e4, 64), (7, 1e3, 2), (12, 3e4, 128)])]
    batch = fq.Batch(specs)
    solo = []
    for i, sp in enumerate(specs):
        _start(batch.instance(i), sp, 10.0)
        s = fq.Solver(**sp)
        s.set_timing(True)
        _start(s, sp, 10.0)
        solo.append(s)
    for n in (150, 350):
        rows = batch.run(n)
        for i, s in enumerate(solo):
            assert rows[i].tobytes() == s.run(n).tobytes(), (n, i)
        _start(batch.instance(1), specs[1], 40.0)
        _start(solo[1], specs[1], 40.0)
    for i, s in enumerate(solo):
        sa, sb = _state(batch.instance(i)), _state(s)
        assert np.array_equal(sa[0], sb[0]) and np.array_equal(sa[1], sb[1])
        s.close()
    batch.close()
