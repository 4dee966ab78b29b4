"""Prefills beside block decodes of one query head per KV head: the planner
takes one launch for both kinds or one for each by the batch's sizes (CPU), and
both ways give the same bits (GPU)."""
import numpy as np
import pytest
import torch

import workloads
from paper_2607_04206_amd import attn
from tests.test_parity import check_cache, check_full
from tests.test_plan import HEADER, parse, plan_of

SEPARATE = HEADER.itemsize  # offset of PlanHeader::separate


def separate(p):
    return int(p.host[SEPARATE:SEPARATE + 4].view(np.int32)[0])


def mix(hq, d, decodes, keys, prefills):
    lens = [int(keys * (0.6 + 0.8 * (k * 7919 % 97) / 97)) for k in range(decodes)]
    return workloads.make_workload("choice", 3, hq=hq, hkv=hq, d=d, decodes=[(n - 64, n) for n in lens], prefills=prefills)


# (heads, head dim, decodes, their mean context, prefills, a launch for each kind), on both sides of each line
SIDES = [(32, 128, 16, 1000, [1819, 1201], 0), (32, 128, 4, 1000, [1819, 1201], 0), (32, 128, 64, 1000, [517, 800, 300], 0),
         # halves past the CUs wait behind short decodes
         (32, 128, 4, 1000, [2048], 1), (32, 128, 16, 1000, [2048], 0), (32, 128, 1, 1000, [2048], 0), (16, 128, 2, 2000, [1541], 0),
         # long contexts in 256-row tiles: full rounds, a half-full last one
         (32, 128, 64, 1000, [8192], 1), (32, 128, 4, 1000, [4480], 0), (16, 128, 1, 1000, [8344], 0), (32, 128, 16, 5000, [8192, 8192], 1),
         # many rounds, little or much to hide
         (32, 128, 4, 1000, [3400] * 8, 1), (32, 128, 64, 1500, [3400] * 6, 0), (32, 128, 4, 1000, [2000] * 8, 0),
         (32, 128, 16, 1000, [8929, 140, 506], 1), (32, 128, 16, 1000, [5216, 140, 506], 0),
         # head dim 64
         (8, 64, 16, 1000, [8192], 1), (8, 64, 4, 1000, [8192], 0), (32, 64, 25, 370, [3419, 3854], 0), (8, 64, 16, 1000, [5741, 5000], 1), (32, 64, 12, 3300, [1329, 1248, 5268, 256], 0),
         (8, 64, 44, 1150, [8162], 1), (8, 64, 41, 4500, [5006], 0), (8, 64, 16, 1000, [2048] * 4, 0)]


@pytest.mark.parametrize("hq,d,decodes,keys,prefills,want", SIDES)
def test_choice(hq, d, decodes, keys, prefills, want):
    p = plan_of(mix(hq, d, decodes, keys, prefills))
    assert p.info.num_prefill_tiles > 0 and p.info.num_decode_tiles > 0
    assert separate(p) == want


@pytest.mark.parametrize("hq,hkv", [(28, 4), (16, 8)])
def test_other_groups_state_no_choice(hq, hkv):
    wl = workloads.make_workload("choice_gqa", 3, hq=hq, hkv=hkv, d=128, decodes=[(64, 900)] * 20, prefills=[2048])
    assert separate(plan_of(wl)) == 0


# the planner's choice, and the other one written into the plan: 512 and fewer halves, more blocks of each kind than CUs
@pytest.mark.gpu
@pytest.mark.parametrize("hq,d,decodes,keys,prefills,force", [(8, 128, 70, 400, [1100, 1025, 1024, 1153], 0), (8, 128, 33, 300, [4200, 1100], 0),
                                                              (8, 128, 5, 300, [1100, 1280], 2), (8, 64, 70, 400, [5200, 97, 500], 0)])
def test_both_ways_give_the_same_bits(hq, d, decodes, keys, prefills, force):
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    dev = torch.device("cuda:0")
    wl = mix(hq, d, decodes, keys, prefills)
    got = []
    for each in (0, 1):
        print(f"[case] {hq}x{d} {decodes} decodes beside {prefills} separate={each}", flush=True)
        p = plan_of(wl, force_kv_splits=force)
        p.host[SEPARATE:SEPARATE + 4] = np.frombuffer(np.int32(each).tobytes(), np.uint8)
        assert parse(p)[0]["n_decode_tiles"] > 0 and separate(p) == each
        t = workloads.device_inputs(wl, dev)
        out, lse = attn.forward(p.to(dev), t["q"], t["k_new"], t["v_new"], t["k_cache"], t["v_cache"], t["page_ids"])
        torch.cuda.synchronize()
        check_cache(wl, t)
        got.append((out, lse))
    check_full(wl, *got[0])
    assert torch.equal(got[0][0].view(torch.int16), got[1][0].view(torch.int16)) and torch.equal(got[0][1], got[1][1])
