"""Resident workgroups that own several buckets and meet more records, or more
addresses, than one pass of their hash takes, against the step kernels: rows
and states bit for bit.  A batch of 130 instances leaves one workgroup for
each, so that one heavy instance is merged by a single workgroup; a partner of
more than 62 address bits keeps every instance at two-word addresses."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SHAPE = dict(lds_slots=2048, block=512, spawn_block=256)
LIGHT = dict(t=1.0, u=1.0, dtau=1e-4, target_walkers=20.0, table_capacity=512, spawn_capacity=4096, buckets=1, **SHAPE)
MOST = 24576  # entries and records of a workgroup that it goes on after


def _start(solver, spec, occ, walkers):
    import paper_2601_19505_amd as fq
    a = fq.encode(occ, spec.get("addr_words", 1))
    solver.set_state([a], [walkers], 0.0, 0, ref=a, yref=10.0)


def _state(solver):
    a, v, shift, step = solver.get_state()
    o = np.lexsort(a.T)
    return a[o], v[o], shift, step


def _occ(spec):
    return [spec["N"] // spec["M"] + (j < spec["N"] % spec["M"]) for j in range(spec["M"])]


def _against_the_step_kernels(spec, walkers, calls, wide):
    """The rows of the heavy instance of a batch, which equal a timed
    solver's, and its state likewise."""
    import paper_2601_19505_amd as fq
    W = 2 if wide else 1
    spec = dict(spec, addr_words=W)
    light = dict(LIGHT, model=spec["model"], M=6, N=6, addr_words=W, lds_slots=spec["lds_slots"], block=spec["block"])
    if spec["model"] == 1 and not wide:
        light.update(M=5, N=5)
    specs = [spec] + [dict(light, seed=i) for i in range(129)]
    if wide:
        specs[1] = dict(light, M=32, N=32, u=0.1)
    batch = fq.Batch(specs)
    solo = fq.Solver(**spec)
    solo.set_timing(True)
    for i, sp in enumerate(specs):
        _start(batch.instance(i), sp, _occ(sp), 10.0 if i else walkers)
    _start(solo, spec, _occ(spec), walkers)
    rows = []
    for n in calls:
        got, want = batch.run(n)[0], solo.run(n)
        for f in want.dtype.names:
            assert np.array_equal(got[f], want[f]), (n, f, int(np.argmax(got[f] != want[f])))
        rows.append(want)
    x, y = _state(batch.instance(0)), _state(solo)
    assert np.array_equal(x[0], y[0]) and np.array_equal(x[1], y[1]) and x[2:] == y[2:]
    batch.close()
    solo.close()
    return np.concatenate(rows)


@pytest.mark.parametrize("buckets", [4, 16])
def test_records_that_cross_the_limit_of_a_pass(buckets):
    """Two words: 16384 items a pass.  About 410 addresses, whose survivors
    stay in registers from step to step, and items that go to and fro across
    that limit."""
    spec = dict(model=0, M=6, N=6, u=4.0, dtau=1e-3, target_walkers=15800.0, seed=11, t_rel=np.inf, buckets=buckets,
                table_capacity=4000, spawn_capacity=40000, **SHAPE)
    print("[batches] records", buckets, flush=True)
    rows = _against_the_step_kernels(spec, 9000.0, (300, 500), wide=True)
    items = rows["len"] + rows["spawns"]
    across = (items[:-1] <= 16384) & (items[1:] > 16384)
    assert np.count_nonzero(across) >= 3 and items.max() < MOST and rows["len"].max() <= 960


@pytest.mark.parametrize("buckets", [4, 16])
@pytest.mark.parametrize("wide, walkers", [(False, 3500.0), (True, 1800.0)])
def test_addresses_that_outgrow_the_hash_in_one_step(wide, walkers, buckets):
    """Walkers on one determinant in momentum space: no more records than the
    first pass of a launch takes, on 361 (358) addresses, whose survivors stay
    in registers; 6676 (4479) addresses meet in the second step, beyond the
    4096 slots of one-word and the 2048 of two-word keys, and the buckets are
    merged again in smaller sets."""
    spec = dict(model=1, M=12, N=12, u=4.0, dtau=8e-3, flags=64, target_walkers=1e5, seed=11, t_rel=np.inf,
                buckets=buckets, table_capacity=7000, spawn_capacity=80000, **SHAPE)
    print("[batches] addresses", wide, buckets, flush=True)
    rows = _against_the_step_kernels(spec, walkers, (2,), wide)
    assert rows["len"][0] <= 960 and rows["len"][0] + rows["spawns"][0] <= MOST
    assert rows["len"][1] > (2048 if wide else 4096)
