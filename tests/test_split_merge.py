"""Split contexts merged by the tile that finishes last (up to seven splits of
every item at four query waves a tile, up to 16 at one) or by the merge launch
(any item above): parity with the oracle at the edges of
both, the same bits whatever the workspace held, and graph replays, whose marks
repeat, over a workspace that nothing clears in between."""
import pytest
import torch

import workloads
from tests.test_parity import check_cache, check_full, run
from tests.test_plan import parse, plan_of


def batch(hq, hkv, d):
    # blocks of 1, 31, 32 and 33 rows (two row blocks), a listed one, 7 to 700 keys past the splits' alignment
    return workloads.make_workload("split_merge", 11, hq=hq, hkv=hkv, d=d, prefills=[],
                                   decodes=[(700, 701, 1), (3, 640, 31), (64, 1025, 32), (17, 1500, 33)],
                                   pos_decodes=[([0, 63, 64, 500, 818], 819)])


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_2607_04206_amd  # noqa: F401
    return torch.device("cuda:0")


@pytest.mark.parametrize("force", [2, 7, 8])
def test_marks_follow_the_partials(force):
    """Every split item's marks (8 bytes per 32 rows, head and split) sit
    after its partials, inside the workspace and apart from the next item's;
    the header field counts them. With an item of more splits than a tile
    merges there are none."""
    wl = batch(28, 4, 128)
    p = plan_of(wl, force_kv_splits=force)
    h, items, *_ = parse(p)
    end, marks = 0, 0
    for it in items[items["num_splits"] > 1]:
        S, n = int(it["num_splits"]), int(it["n"])
        assert int(it["ws_o"]) >= end
        at = int(it["ws_lse"]) + -(-S * n * 28 // 64) * 64
        size = -(-(-(-n // 32) * 28 * S * 2) // 64) * 64 if force <= 7 else 0
        end, marks = at + size, marks + size
    assert int(h["reserved"]) == 4 * marks and end * 4 == p.workspace_bytes


@pytest.mark.gpu
@pytest.mark.parametrize("hq,hkv,d", [(4, 4, 64), (4, 4, 128), (4, 2, 128), (28, 4, 128), (8, 4, 64), (16, 1, 128)])
@pytest.mark.parametrize("force", [2, 7, 8, 14, 16, 17])
def test_merged_rows(dev, hq, hkv, d, force):
    from paper_2607_04206_amd import attn
    wl = batch(hq, hkv, d)
    p, t, out, lse = run(wl, dev, force_splits=force)
    check_full(wl, out, lse)
    check_cache(wl, t)
    args = (p, t["q"], t["k_new"], t["v_new"], t["k_cache"], t["v_cache"], t["page_ids"])
    for fill in (0, 0x5A, 0xFF):
        ws = torch.full((p.workspace_bytes,), fill, dtype=torch.uint8, device=dev)
        for _ in range(2):  # the second call finds the first one's partials
            out2, lse2 = attn.forward(*args, workspace=ws)
            assert torch.equal(out2.view(torch.int16), out.view(torch.int16)) and torch.equal(lse2, lse)


@pytest.mark.gpu
def test_replays_over_an_uncleared_workspace(dev):
    from paper_2607_04206_amd import attn
    wl = batch(8, 4, 128)
    p, t, out0, lse0 = run(wl, dev, force_splits=5)
    args = (p, t["q"], t["k_new"], t["v_new"], t["k_cache"], t["v_cache"], t["page_ids"])
    ws = torch.empty((p.workspace_bytes,), dtype=torch.uint8, device=dev)
    out, lse = torch.empty_like(out0), torch.empty_like(lse0)
    attn.forward(*args, out=out, lse=lse, workspace=ws)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        attn.forward(*args, out=out, lse=lse, workspace=ws)
    for r in range(6):
        out.fill_(float("nan"))
        lse.fill_(float("nan"))
        g.replay()
        if r % 2:
            g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int16), out0.view(torch.int16)) and torch.equal(lse, lse0), f"replay {r}"
        if r % 3 == 2:  # another call's marks in the same workspace
            attn.forward(*args, workspace=ws)


@pytest.mark.gpu
def test_two_streams_at_once(dev):
    """Calls of one plan in flight on two streams, each with its own workspace."""
    from paper_2607_04206_amd import attn
    wl = batch(28, 4, 128)
    p, t, out0, lse0 = run(wl, dev, force_splits=8)
    args = (p, t["q"], t["k_new"], t["v_new"], t["k_cache"], t["v_cache"], t["page_ids"])
    streams = [torch.cuda.Stream(dev) for _ in range(2)]
    bufs = [(torch.empty_like(out0), torch.empty_like(lse0), torch.empty((p.workspace_bytes,), dtype=torch.uint8, device=dev))
            for _ in streams]
    torch.cuda.synchronize()
    for _ in range(20):
        for s, (o, l, ws) in zip(streams, bufs):
            attn.forward(*args, out=o, lse=l, workspace=ws, stream=s)
    torch.cuda.synchronize()
    for o, l, _ in bufs:
        assert torch.equal(o.view(torch.int16), out0.view(torch.int16)) and torch.equal(l, lse0)
