"""Prefill-shaped tiles and block decodes of one query head per KV head in one
launch: more tiles of each kind than one round of CUs, more of one than of the
other, 256-row tiles taken in halves (the last half past the rows), listed
rows, a cached block of more than 32 rows, split contexts."""
import pytest
import torch

import workloads
from tests.test_parity import check_cache, check_full, check_pool_untouched, run

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_2607_04206_amd  # noqa: F401
    return torch.device("cuda:0")


# (decodes, prefill lengths) by tiles of 8 heads: 560 decodes, 320 halves of
# 256-row tiles; 1 decode; 584 decodes beside one short prefill; 24 beside 640
MIXES = {"both": (70, (1100, 1025, 1024, 1153)), "one decode": (1, (1100,)), "decodes": (73, (97,)),
         "prefills": (3, (1100, 2000, 1024, 1024, 1100, 1030))}


@pytest.mark.parametrize("mix,d,force", [(mix, d, force) for mix in ("both", "one decode", "decodes")
                                         for d, force in ((64, 0), (128, 0), (128, 2))] + [("prefills", 128, 0)])
def test_mixed_launch(dev, mix, d, force):
    count, prefills = MIXES[mix]
    dec = [(7 * k % 90, 130 + 11 * k) for k in range(count)]
    wl = workloads.make_workload("mixed", 17, hq=8, hkv=8, d=d, decodes=dec + [(37, 3000, 1030)], prefills=list(prefills),
                                 pos_decodes=[([0, 15, 16, 99, 170], 171)])
    p, t, out, lse = run(wl, dev, force_splits=force)
    assert p.info.num_prefill_tiles > 0 and p.info.num_decode_tiles > 0
    check_full(wl, out, lse)
    check_cache(wl, t)
    check_pool_untouched(wl, t)

