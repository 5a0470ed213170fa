"""The finalize kernel by several workgroups (from 2048 buckets on) against
one workgroup: the rows do not depend on the bucket count."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SPEC = dict(model=0, M=9, N=9, u=4.0, dtau=1e-3, target_walkers=3e3, seed=21)


def _run(buckets, **more):
    import paper_2601_19505_amd as fq
    s = fq.Solver(**dict(SPEC, buckets=buckets, table_capacity=max(12000, 2 * buckets),
                         spawn_capacity=max(60000, 20 * buckets), **more))
    s.set_timing(True)  # step kernels
    a = fq.start_address(0, 9, 9, more.get("addr_words", 1))
    s.set_state([a], [20.0], 0.0, 0, ref=a, yref=10.0)
    rows = [s.run(n) for n in (1, 200, 300)]
    s.close()
    return np.concatenate(rows)


@pytest.mark.parametrize("buckets", [1024, 2048, 4096, 16384, 32768])
def test_rows_do_not_depend_on_the_finalize_workgroups(buckets):
    for more in (dict(), dict(addr_words=2, flags=32)):
        print("[finalize]", buckets, more, flush=True)
        assert _run(buckets, **more).tobytes() == _run(16, **more).tobytes()
