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


@pytest.mark.parametrize("d,prefills,force", [(128, (1100, 1025, 1024, 1153), 1), (128, (1100, 1280), 2), (128, (97, 1100), 1), (64, (1100, 300), 1)])
def test_rows_are_those_of_a_launch_of_their_own(dev, d, prefills, force):
    """A prefill's bits (and those of a cached block of more than 32 rows) do
    not depend on the block decodes beside it: 256-row tiles keep their
    128-key stages when they are taken in halves. Nor do a decode's."""
    from paper_2607_04206_amd import attn
    dec = [(7 * k, 130 + 11 * k) for k in range(20)]
    wl = workloads.make_workload("mixed_bits", 23, hq=8, hkv=8, d=d, decodes=dec + [(37, 3000, 1030)], prefills=list(prefills))
    p, t, out, lse = run(wl, dev, force_splits=force)
    splits = [len(p.item_splits(i)) - 1 for i in range(wl.num_items)]
    for lo, hi in ((0, len(dec)), (len(dec), wl.num_items)):
        r0, r1 = int(wl.q_indptr[lo]), int(wl.q_indptr[hi])
        g0, g1 = int(wl.page_indptr[lo]), int(wl.page_indptr[hi])
        alone = attn.plan(q_indptr=wl.q_indptr[lo:hi + 1] - r0, q_offset=wl.q_offset[lo:hi], kv_len=wl.kv_len[lo:hi],
                          page_indptr=wl.page_indptr[lo:hi + 1] - g0, page_ids=wl.page_ids[g0:g1], num_q_heads=8, num_kv_heads=8,
                          head_dim=d, num_pool_pages=wl.num_pool_pages, sm_scale=wl.sm_scale, force_kv_splits=force,
                          device=dev)
        assert [len(alone.item_splits(i)) - 1 for i in range(hi - lo)] == splits[lo:hi]
        assert (alone.info.num_prefill_tiles > 0) != (alone.info.num_decode_tiles > 0)
        out1, lse1 = attn.forward(alone, t["q"][r0:r1], t["k_new"][r0:r1], t["v_new"][r0:r1], t["k_cache"], t["v_cache"],
                                  t["page_ids"][g0:g1])
        assert torch.equal(out1.view(torch.int16), out[r0:r1].view(torch.int16)) and torch.equal(lse1, lse[r0:r1]), (lo, hi)
