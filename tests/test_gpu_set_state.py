"""Checks of a state's entries on the device: what is refused, the entry that
the error names, and that a refused call leaves the state as it was."""
import numpy as np
import pytest

import synthetic

pytestmark = pytest.mark.gpu

SPEC = dict(model=0, M=9, N=9, u=4.0, dtau=1e-3, target_walkers=2e3, seed=5, table_capacity=9000,
            spawn_capacity=60000)


def _fq():
    import paper_2601_19505_amd as fq
    return fq


def _entries(n, W):
    fq = _fq()
    rng = np.random.default_rng(3)
    occ = synthetic.random_occupations(rng, SPEC["M"], SPEC["N"], n)
    return fq.encode_many(occ, W), synthetic.random_amplitudes(rng, n, hi=20.0)


def _sorted(solver):
    a, v, shift, step = solver.get_state()
    o = np.lexsort(a.T)
    return a[o].tobytes(), v[o].tobytes(), shift, step


BROKEN = {
    "duplicate, neighbours": (lambda a, v: a.__setitem__(51, a[50]), "duplicate address in state"),
    "duplicate, first and last": (lambda a, v: a.__setitem__(len(a) - 1, a[0]), "duplicate address in state"),
    "a boson too many": (lambda a, v: a.__setitem__((700, 0), a[700, 0] | (~a[700, 0] & (~a[700, 0] + np.uint64(1)))),
                         "at entry 700"),
    "a bit beyond the address": (lambda a, v: a.__setitem__((3, 0), (a[3, 0] & (a[3, 0] - np.uint64(1)))
                                                           | np.uint64(1 << 17)), "at entry 3"),
    "no boson": (lambda a, v: a.__setitem__((5, 0), np.uint64(0)), "at entry 5"),
    "zero value": (lambda a, v: v.__setitem__(900, 0.0), "at entry 900"),
    "nan": (lambda a, v: v.__setitem__(1, np.nan), "at entry 1"),
    "infinite, and a later zero": (lambda a, v: (v.__setitem__(20, -np.inf), v.__setitem__(30, 0.0)), "at entry 20"),
}


@pytest.mark.parametrize("W", [1, 2])
@pytest.mark.parametrize("buckets", [1, 8, 256])
def test_refused_states_are_named_and_leave_the_state(W, buckets):
    fq = _fq()
    s = fq.Solver(addr_words=W, buckets=buckets, **SPEC)
    twin = fq.Solver(addr_words=W, buckets=buckets, **SPEC)
    a, v = _entries(1000, W)
    for x in (s, twin):
        x.set_state(a, v, 0.0, 0, ref=a[0])
        x.run(7)  # an odd number: the state lies in the second table
    for name, (spoil, says) in BROKEN.items():
        print("[set_state]", name, flush=True)
        b, w = a.copy(), v.copy()
        spoil(b, w)
        with pytest.raises(fq.FqError) as e:
            s.set_state(b, w, 1.0, 3, ref=a[0])
        assert e.value.status == -1 and says in str(e.value), (name, str(e.value))
        assert _sorted(s) == _sorted(twin), name
    assert s.run(20).tobytes() == twin.run(20).tobytes()
    # and a sound one replaces it, whichever table the old one lies in
    for k in (0, 1, 2):
        s.run(k)
        s.set_state(a, v, 0.5, 40, ref=a[0])
        fresh = fq.Solver(addr_words=W, buckets=buckets, **SPEC)
        fresh.set_state(a, v, 0.5, 40, ref=a[0])
        assert _sorted(s) == _sorted(fresh)
        assert s.run(15).tobytes() == fresh.run(15).tobytes()
        fresh.close()
    s.close()
    twin.close()


def test_a_state_beyond_the_capacity_is_refused_after_its_entries_are_checked():
    fq = _fq()
    spec = dict(SPEC, table_capacity=300, spawn_capacity=300)
    s = fq.Solver(buckets=1, **spec)
    a, v = _entries(4000, 1)
    with pytest.raises(fq.FqError) as e:
        s.set_state(a, v, 0.0, 0, ref=a[0])
    assert e.value.status == -2
    v[3000] = 0.0
    with pytest.raises(fq.FqError) as e:
        s.set_state(a, v, 0.0, 0, ref=a[0])
    assert e.value.status == -1 and "at entry 3000" in str(e.value)
    s.close()
