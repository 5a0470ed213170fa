"""The arrays of a state are its own: no larger buffer stays behind them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W", [1, 2])
@pytest.mark.parametrize("cap", [None, 3, 10**6])
def test_a_state_owns_no_more_than_its_entries(W, cap):
    import paper_2601_19505_amd as fq
    s = fq.Solver(model=0, M=8, N=8, u=4.0, target_walkers=100.0, seed=3, addr_words=W, table_capacity=200000,
                  spawn_capacity=200000)
    a = fq.start_address(0, 8, 8, W)
    s.set_state([a], [10.0], 0.0, 0, ref=a, yref=10.0)
    n = int(s.run(200)["len"][-1])
    assert n > 3
    addrs, vals, _, step = s.get_state(cap)
    assert addrs.shape == (n, W) and vals.shape == (n,) and step == 200
    for x in (addrs, vals):
        assert x.base is None and x.flags.owndata and x.flags.c_contiguous and x.flags.writeable
    again = s.get_state()
    o, q = np.lexsort(addrs.T), np.lexsort(again[0].T)
    assert np.array_equal(addrs[o], again[0][q]) and np.array_equal(vals[o], again[1][q])
    s.close()


def test_states_after_every_way_to_a_new_one():
    """Run, set, copied, stepped by a batch, failed: as many entries as there
    are, and no error left behind."""
    import paper_2601_19505_amd as fq
    spec = dict(model=0, M=8, N=8, u=4.0, target_walkers=200.0, seed=3, table_capacity=2000, spawn_capacity=20000,
                buckets=1, lds_slots=1024, block=256)
    a = fq.start_address(0, 8, 8)
    s, t, b = fq.Solver(**spec), fq.Solver(**spec), fq.Batch([spec, spec])
    for x in (s, t, b.instance(0), b.instance(1)):
        x.set_state([a], [10.0], 0.0, 0, ref=a, yref=10.0)
    assert len(s.get_state()[1]) == 1
    n = int(s.run(150)["len"][-1])
    assert len(s.get_state()[1]) == n
    t.copy_state_from(s)
    assert len(t.get_state()[1]) == n
    s.set_state([a], [10.0], 0.0, 0, ref=a, yref=10.0)
    assert len(s.get_state()[1]) == 1
    assert len(b.instance(0).get_state()[1]) == 1
    b.instance(0).run(50)
    k = int(b.run(100)[0]["len"][-1])
    assert len(b.instance(0).get_state()[1]) == k and b.instance(0).last_error() == ""
    # a run that fails leaves the state of its last step
    grow = fq.Solver(**dict(spec, target_walkers=1e5))
    grow.set_state([a], [10.0], 0.0, 0, ref=a, yref=10.0)
    grow.run(20)
    with pytest.raises(fq.FqError) as e:
        grow.run(2000)
    rows = e.value.stats[e.value.stats["step"] > 0]
    assert len(grow.get_state()[1]) == int(rows["len"][-1])
    for x in (s, t, b, grow):
        x.close()
