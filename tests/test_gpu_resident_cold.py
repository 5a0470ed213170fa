"""Short runs on many workgroups whose data has been driven out of the caches
in between, against one long run and the step kernels: what a workgroup wrote
before the barrier has to be there for all others behind it, however long its
way to memory is."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# 256 workgroups on all XCDs; records of 12 and of 16 bytes
SPECS = {
    "27 bits": dict(model=0, M=14, N=14, u=6.0, dtau=1e-3, target_walkers=2.6e5, seed=61),
    "37 bits": dict(model=0, M=19, N=19, u=4.0, dtau=1e-3, target_walkers=2.0e5, seed=86),
}


def _solver(spec):
    import paper_2601_19505_amd as fq
    s = fq.Solver(table_capacity=320000, spawn_capacity=720000, buckets=512, lds_slots=2048, block=512, spawn_block=256,
                  **spec)
    a = fq.start_address(spec["model"], spec["M"], spec["N"])
    s.set_state([a], [10.0], 0.0, 0, ref=a, yref=10.0)
    return s


@pytest.mark.parametrize("name", list(SPECS))
def test_short_runs_from_cold_caches_equal_a_long_one(name):
    import torch
    print("[cold]", name, flush=True)
    ramp, per, calls = 1200, 3, 3000
    short, long, kernels = (_solver(SPECS[name]) for _ in range(3))
    kernels.set_timing(True)
    for s in (short, long, kernels):
        s.run(ramp)
    want = long.run(per * calls)
    assert kernels.run(300).tobytes() == want[:300].tobytes()
    other = torch.zeros(1 << 28, device="cuda")  # 1 GiB
    for k in range(calls):
        other.add_(1.0)
        got = short.run(per)
        assert got.tobytes() == want[per * k: per * (k + 1)].tobytes(), (k, got, want[per * k: per * (k + 1)])
    for s in (short, long, kernels):
        s.close()
