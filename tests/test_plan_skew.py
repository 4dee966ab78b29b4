"""GQA decode batches with nearly as many contexts as CUs hold work-groups: a
long context among short ones is cut, equal contexts are not."""
import numpy as np
import pytest
import torch

import workloads
from tests.test_parity import check_cache, check_full, run
from tests.test_plan import parse, plan_of


def batch(hq, hkv, d, count, long):
    dec = [(64, 300 + 7 * k % 200) for k in range(count - 1)] + [(1000, long)]
    return workloads.make_workload("plan_skew", 5, hq=hq, hkv=hkv, d=d, prefills=[], decodes=dec)


# 252 or 248 whole-group tiles of the 256 that the CUs hold; the long context alone is cut
@pytest.mark.parametrize("hq,hkv,d,count", [(28, 4, 128, 63), (32, 8, 128, 31), (32, 8, 64, 31), (6, 2, 64, 127)])
@pytest.mark.parametrize("long,cut", [(4000, True), (1040, False)])
def test_long_context_is_cut(hq, hkv, d, count, long, cut):
    wl = batch(hq, hkv, d, count, long)
    if not cut:
        wl = workloads.make_workload("plan_even", 5, hq=hq, hkv=hkv, d=d, prefills=[], decodes=[(64, long)] * count)
    h, items, *_ = parse(plan_of(wl))
    assert (items["num_splits"][:-1] == 1).all()
    assert (int(items["num_splits"][-1]) > 2) == cut  # one more tile per KV head would fit without more rounds
    lens = items["split_len"].astype(np.int64) * items["num_splits"]
    assert (lens >= items["L"]).all()


def test_cut_stays_within_the_scratch():
    """Contexts of which many gain by a cut beyond the slots: never more partials
    than the allocation-free forward holds (without the limit 19 of these
    batches, and up to 1.98 times as many)."""
    from paper_2607_04206_amd._lib import lib
    rng = np.random.default_rng(3)
    beyond = 0
    for _ in range(60):
        count = int(rng.integers(20, 32))
        lens = np.exp(rng.normal(np.log(3000), 1.0, count)).astype(int) + 600
        wl = workloads.make_workload("plan_scratch", 5, hq=64, hkv=8, d=128, prefills=[],
                                     decodes=[(64, int(min(n, 7000))) for n in lens])
        p = plan_of(wl)
        h, items, *_ = parse(p)
        assert len(items) == count
        beyond += p.info.num_decode_tiles > 256
        assert p.workspace_bytes - int(h["reserved"]) <= int(lib.sangam_noalloc_scratch_bytes())
    assert beyond > 20


@pytest.mark.gpu
@pytest.mark.parametrize("hq,hkv,d,count", [(28, 4, 128, 63), (6, 2, 64, 127)])
def test_cut_batch_matches(hq, hkv, d, count):
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    wl = batch(hq, hkv, d, count, 4000)
    p, t, out, lse = run(wl, torch.device("cuda:0"))
    assert p.info.max_splits > 2
    check_full(wl, out, lse)
    check_cache(wl, t)
