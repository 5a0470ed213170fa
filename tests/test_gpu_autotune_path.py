"""fq_autotune times what fq_run does: an instance that takes many steps in one
launch is timed so, and a layout that keeps it from that is not preferred."""
import time

import pytest

pytestmark = pytest.mark.gpu


def test_trials_take_the_kernels_of_a_run():
    import torch

    import paper_2601_19505_amd as fq
    s = fq.Solver(model=0, M=8, N=8, u=4.0, dtau=1e-3, target_walkers=2e3, seed=11, table_capacity=8192,
                  spawn_capacity=40000, buckets=8)
    a = fq.start_address(0, 8, 8)
    s.set_state([a], [10.0], 0.0, 0, ref=a, yref=10.0)
    s.run(1500)
    steps = 1000
    ms, best = s.autotune([dict(buckets=8), dict(buckets=16384)], trial_steps=steps)
    took = []
    for _ in range(4):
        torch.cuda.synchronize()
        t = time.perf_counter()
        s.run(steps)
        took.append((time.perf_counter() - t) * 1e3 / steps)
    print("[autotune]", ms, best, took, flush=True)
    # (the step kernels take 45 us a step, many steps in one launch 11)
    assert best == 0 and 0.5 * min(took) < ms[0] < 1.7 * min(took) and ms[1] > 2.0 * ms[0]
    s.close()
