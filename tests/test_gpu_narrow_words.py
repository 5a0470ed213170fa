"""Two-word addresses of at most 62 bits are kept in one word by a solver or a
batch of such instances, and in two beside wider instances or with dumps: the
same rows and states, states that pass between the two, and what was refused."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

RING = dict(model=0, M=8, N=8, u=4.0, dtau=1e-3, target_walkers=2e3, seed=31, addr_words=2, table_capacity=8192,
            spawn_capacity=40000, buckets=8, lds_slots=2048, block=512, spawn_block=256)
WIDE = dict(RING, M=33, N=33, u=0.1, target_walkers=200.0, seed=5)  # 65 address bits
CASES = {
    "ring": RING,
    "62 bits": dict(RING, M=31, N=32, u=0.2, target_walkers=1e3),
    "ring, initiator": dict(RING, initiator=3.0),
    "ring, 32 bits, initiator": dict(RING, M=16, N=17, u=0.5, initiator=3.0),
    "lattice": dict(RING, model=2, M=12, N=12, lx=4, t=0.1, u=1.0, g=0.5, dtau=5e-3),
    "lattice, 128 buckets": dict(RING, model=2, M=12, N=12, lx=4, t=0.1, u=1.0, g=0.5, dtau=5e-3, buckets=128,
                                 table_capacity=20000, spawn_capacity=100000),
}
DUMPS = 1  # FQ_FLAG_DUMP_SPAWNS: the kernels keep both words


def _start(s, sp, walkers=10.0):
    import paper_2601_19505_amd as fq
    a = fq.start_address(sp["model"], sp["M"], sp["N"], 2)
    s.set_state([a], [walkers], 0.0, 0, ref=a, yref=10.0)


def _state(s):
    a, v, shift, step = s.get_state()
    assert a.shape[1] == 2
    o = np.lexsort(a.T)
    return a[o], v[o], shift, step


def _equal(x, y):
    return np.array_equal(x[0], y[0]) and np.array_equal(x[1], y[1]) and x[2:] == y[2:]


@pytest.mark.parametrize("kernels", [False, True])
@pytest.mark.parametrize("name", list(CASES))
def test_one_word_equals_two(name, kernels):
    import paper_2601_19505_amd as fq
    sp = CASES[name]
    print("[narrow]", name, kernels, flush=True)
    wide = dict(WIDE, initiator=sp.get("initiator"), model=sp["model"])
    if sp["model"] == 2:
        wide.update(M=36, N=36, lx=6, t=0.1, u=1.0, g=0.5)
    solo = fq.Solver(**sp)
    pair = fq.Batch([sp, wide])       # two words, for the second instance
    both = fq.Batch([sp, dict(sp, seed=77)])  # one word
    for b, second in ((pair, wide), (both, sp)):
        _start(b.instance(0), sp)
        _start(b.instance(1), second)
        if kernels:
            b.instance(0).set_timing(True)
    _start(solo, sp)
    if kernels:
        solo.set_timing(True)
    for n in (1, 150, 250):
        rows = solo.run(n)
        assert rows.tobytes() == pair.run(n)[0].tobytes() == both.run(n)[0].tobytes(), n
    assert _equal(_state(solo), _state(pair.instance(0))) and _equal(_state(solo), _state(both.instance(0)))
    # states pass between the two widths
    x, y = fq.Solver(**sp), fq.Batch([sp, wide])
    _start(x, sp, 3.0)
    _start(y.instance(0), sp, 3.0)
    _start(y.instance(1), wide)
    x.copy_state_from(pair.instance(0))
    y.instance(0).copy_state_from(solo)
    assert _equal(_state(x), _state(solo)) and _equal(_state(y.instance(0)), _state(solo))
    rows = solo.run(60)
    assert rows.tobytes() == x.run(60).tobytes() == y.run(60)[0].tobytes()
    for s in (solo, x, pair, both, y):
        s.close()


def test_dumps_and_refusals_keep_two_words():
    import paper_2601_19505_amd as fq
    s, d = fq.Solver(**RING), fq.Solver(**dict(RING, flags=DUMPS))
    _start(s, RING)
    _start(d, RING)
    assert s.run(100).tobytes() == d.run(100).tobytes()
    assert _equal(_state(s), _state(d))
    before = _state(s)
    for a1 in (1, 1 << 63):
        bad = before[0].copy()
        bad[-1, 1] = a1
        with pytest.raises(fq.FqError) as e:
            s.set_state(bad, before[1], 0.0, 0, ref=before[0][0], yref=1.0)
        assert e.value.status == -1 and "entry %d" % (len(bad) - 1) in str(e.value)
        with pytest.raises(fq.FqError):
            s.set_state(before[0], before[1], 0.0, 0, ref=bad[-1], yref=1.0)
    assert _equal(_state(s), before)
    s.close()
    d.close()
    # workspaces and limits are those of two words
    with pytest.raises(fq.FqError):
        fq.Solver(**dict(RING, lds_slots=8192, block=1024))


def test_momentum_addresses_around_31_bits_share_a_batch():
    """Their one-word kernels differ, so the batch keeps two words."""
    import paper_2601_19505_amd as fq
    mom = dict(RING, model=1, u=1.0, dtau=5e-4, table_capacity=40000, spawn_capacity=200000, target_walkers=1e3)
    specs = [dict(mom, M=9, N=9), dict(mom, M=18, N=18, seed=32)]
    b = fq.Batch(specs)
    solo = [fq.Solver(**sp) for sp in specs]
    for i, sp in enumerate(specs):
        _start(b.instance(i), sp)
        _start(solo[i], sp)
    rows = b.run(200)
    for i in range(2):
        assert rows[i].tobytes() == solo[i].run(200).tobytes(), i
        solo[i].close()
    b.close()
