"""The planner's search for a decode chunk runs only where the chunk is read.
It walks the chip's CUs, so a plan that does not read it takes as long for a
chip of a million times as many. Runs without a GPU."""
import time

import numpy as np
import pytest

import workloads
from tests.test_plan import plan_of


def best_of(n, wl, **kw):
    times = []
    for _ in range(n):
        t = time.perf_counter()
        p = plan_of(wl, **kw)
        times.append(time.perf_counter() - t)
    return min(times), p


@pytest.mark.parametrize("prefills,kw", [([200], {}), ([], dict(force_kv_splits=1)), ([], dict(force_kv_splits=3))])
def test_no_search_whose_chunk_is_not_read(prefills, kw):
    wl = workloads.make_workload("plan_cost", 5, hq=28, hkv=4, d=128, prefills=prefills,
                                 decodes=[(64, 300 + 37 * k) for k in range(40)])
    small, p = best_of(15, wl, num_cus=256, **kw)
    large, q = best_of(15, wl, num_cus=1 << 24, **kw)
    if prefills:  # (forced splits of decodes alone take other tiles on a chip that they would not fill)
        assert p.info.num_fused_decode_tiles == 40 * 4 * 2 and np.array_equal(p.host[256:], q.host[256:])  # the headers state the CUs
    assert large < 5 * small + 1e-3, (small, large)
