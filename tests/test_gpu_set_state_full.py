"""States that do not fit: entries that fill a bucket leave the state that is
there as it is, from the host and from another handle; a state whose spawns do
not fit cannot be stepped, and no row of it is reported."""
import numpy as np
import pytest

import synthetic

pytestmark = pytest.mark.gpu

# 73 entries a bucket, 4672 in all
SPEC = dict(model=0, M=9, N=9, u=4.0, dtau=1e-3, target_walkers=30.0, seed=5, table_capacity=64, spawn_capacity=20000,
            buckets=64)


def _state(solver):
    a, v, shift, step = solver.get_state()
    o = np.lexsort(a.T)
    return a[o].tobytes(), v[o].tobytes(), shift, step


def _entries(n, W):
    import paper_2601_19505_amd as fq
    rng = np.random.default_rng(3)
    return (fq.encode_many(synthetic.random_occupations(rng, SPEC["M"], SPEC["N"], n), W),
            synthetic.random_amplitudes(rng, n, lo=0.5, hi=1.0, heavy=0.0))


@pytest.mark.parametrize("W", [1, 2])
@pytest.mark.parametrize("steps", [0, 1, 4])
def test_a_full_bucket_leaves_the_state(W, steps):
    import paper_2601_19505_amd as fq
    s, twin = (fq.Solver(addr_words=W, **SPEC) for _ in range(2))
    a, v = _entries(4400, W)  # 69 a bucket on average: some get more than 73
    small = a[:40], v[:40]
    for x in (s, twin):
        x.set_state(*small, 0.0, 0, ref=a[0])
        x.run(steps)
    print("[set_state] full", W, steps, flush=True)
    with pytest.raises(fq.FqError) as e:
        s.set_state(a, v, 2.0, 1000, ref=a[1])
    assert e.value.status == -2 and "table bucket capacity" in str(e.value)
    assert _state(s) == _state(twin)
    # the same from a handle whose buckets hold them
    roomy = fq.Solver(addr_words=W, **dict(SPEC, table_capacity=4096))
    with pytest.raises(fq.FqError) as e:
        s.copy_state_from(roomy)
    assert e.value.status == -1
    roomy.set_state(a, v, 2.0, 1000, ref=a[1])
    with pytest.raises(fq.FqError) as e:
        s.copy_state_from(roomy)
    assert e.value.status == -2
    assert _state(s) == _state(twin)
    assert s.run(25).tobytes() == twin.run(25).tobytes() and _state(s) == _state(twin)
    for x in (s, twin, roomy):
        x.close()


def test_a_full_bucket_leaves_no_state_where_there_was_none():
    import paper_2601_19505_amd as fq
    s = fq.Solver(**SPEC)
    a, v = _entries(4400, 1)
    with pytest.raises(fq.FqError) as e:
        s.set_state(a, v, 0.0, 0, ref=a[0])
    assert e.value.status == -2
    for call in (lambda: s.run(1), s.get_state):
        with pytest.raises(fq.FqError) as e:
            call()
        assert e.value.status == -1
    s.set_state(a[:40], v[:40], 0.0, 0, ref=a[0])
    assert s.run(3)["step"][-1] == 3
    s.close()


@pytest.mark.parametrize("batch", [False, True])
@pytest.mark.parametrize("steps", [0, 3])
def test_spawns_that_do_not_fit(steps, batch):
    """Every column exact: 300 entries have 2816 spawns, in a slab for
    1090.  The state that was there was at step `steps`, the new one is
    at 1000: a run must not take the difference for steps that it made."""
    import paper_2601_19505_amd as fq
    spec = dict(SPEC, table_capacity=800, spawn_capacity=800, buckets=1, t_rel=0.0, target_walkers=20.0)
    b = fq.Batch([spec, dict(spec, seed=6)]) if batch else None
    s = b.instance(0) if batch else fq.Solver(**spec)
    run = b.run if batch else s.run
    a, v = _entries(300, 1)
    few = a[:2], np.array([1.5, -1.0])
    s.set_state(*few, 0.0, 0, ref=a[0])
    if batch:
        b.instance(1).set_state(*few, 0.0, 0, ref=a[0])
    run(steps)
    print("[set_state] spawns", steps, batch, flush=True)
    with pytest.raises(fq.FqError) as e:
        s.set_state(a, v, 0.0, 1000, ref=a[0])
    assert e.value.status == -2 and "spawn slab" in str(e.value)
    with pytest.raises(fq.FqError) as e:
        run(2)
    assert e.value.status == -2
    rows = e.value.stats[0] if batch else e.value.stats
    assert rows.shape == (2,) and not rows["step"].any()
    assert s.get_state()[3] == 1000
    # another state, and all is well
    fresh = fq.Solver(**spec)
    for x in (s, fresh):
        x.set_state(*few, 0.0, 7, ref=a[0])
    got = run(2)
    assert (got[0] if batch else got).tobytes() == fresh.run(2).tobytes()
    fresh.close()
    (b or s).close()
