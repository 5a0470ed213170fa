"""States that do not fit: entries that fill a bucket leave the state that is
there as it is, from the host and from another handle."""
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
