"""Which launches a forward makes (sangam_plan_launches), and what is made of
it: bench.py counts a launch's work and time by it."""
import ctypes

import numpy as np
import pytest
import torch

import bench
import workloads
from paper_2607_04206_amd import attn
from paper_2607_04206_amd._lib import lib
from tests.test_parity import check_full
from tests.test_plan import plan_of


def mix(hq, hkv, decodes, prefills, d=128):
    return workloads.make_workload("launches", 3, hq=hq, hkv=hkv, d=d, decodes=decodes, prefills=prefills)


SHARED = lambda: mix(32, 32, [(64, 1000)] * 16, [1819, 1201])  # noqa: E731
CASES = [(SHARED, {}, (True, False, False)),  # MHA: both kinds in one launch
         (lambda: mix(32, 32, [(64, 1000)] * 4, [2048]), {}, (True, True, False)),  # two are faster; splits merged by the tiles
         (lambda: mix(28, 4, [(64, 1000)] * 16, [1819]), {}, (True, False, False)),  # block decodes fused
         (lambda: mix(16, 8, [(64, 1000)] * 16, [1819]), {}, (True, True, False)),
         (lambda: mix(8, 8, [(64, 2000)], []), dict(force_kv_splits=4), (False, True, False)),
         (lambda: mix(8, 8, [(64, 2000)], []), dict(force_kv_splits=32), (False, True, True)),
         (lambda: mix(8, 8, [(64, 2000)], [200]), dict(force_kv_splits=32), (True, False, True))]


@pytest.mark.parametrize("make,kw,want", CASES)
def test_launches(make, kw, want):
    p = plan_of(make(), **kw)
    assert p.launches() == want


def test_errors():
    p = plan_of(SHARED())
    assert lib.sangam_plan_launches(None, (ctypes.c_int32 * 3)()) == -8
    assert lib.sangam_plan_launches(p.host_ptr(), None) == -1


@pytest.mark.parametrize("make", [SHARED, CASES[1][0], CASES[2][0]])
def test_the_launches_hold_the_call_s_work(make):
    wl = make()
    ran = dict(zip(bench.PHASES, plan_of(wl).launches()))
    work = bench.split_work(wl, decodes_in_prefill=not ran["decode_attn"])
    assert np.isclose(sum(work[k][0] for k in work if ran[k]), wl.flops())
    assert all(ran[k] or work[k] == (0.0, 0.0) for k in work)


@pytest.mark.gpu
@pytest.mark.parametrize("k", [0, 1, 6])
def test_events_of_the_launches_that_ran(k):
    """The timed entry point gives the plain one's bits and a positive time for
    each launch that ran."""
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    dev = torch.device("cuda:0")
    make, kw, want = CASES[k]
    wl = make()
    t = workloads.device_inputs(wl, dev)
    p = plan_of(wl, device=dev, **kw)
    args = (p, t["q"], t["k_new"], t["v_new"], t["k_cache"], t["v_cache"], t["page_ids"])
    out0, lse0 = attn.forward(*args)
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(6)]
    for e in ev:
        e.record()
    for _ in range(3):
        out, lse = attn.forward(*args, launch_events=ev)
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), out0.view(torch.int16)) and torch.equal(lse, lse0)
    for j, ran in enumerate(want):
        assert ev[2 * j].elapsed_time(ev[2 * j + 1]) > 0.0 or not ran
    check_full(wl, out, lse)
