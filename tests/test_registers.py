"""Registers of the built kernels: none spills vector registers, and the decode
tiles of five to eight query heads at head dim 64 leave room for four waves per
SIMD, so that a CU holds two or three of them (CPU). Their merges of as many
splits as a tile takes, and of one more (GPU)."""
import os
import re
import shutil
import subprocess

import pytest
import torch

import workloads
from paper_2607_04206_amd import _lib
from tests.test_parity import check_cache, check_full, run

LLVM = "/opt/rocm/llvm/bin/"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if not os.path.exists(LLVM + "llvm-readelf"):
        pytest.skip("needs llvm-readelf")
    d = str(tmp_path_factory.mktemp("registers"))
    shutil.copy(_lib.LIB_PATH, d)
    subprocess.run([LLVM + "llvm-objdump", "--offloading", os.path.basename(_lib.LIB_PATH)], cwd=d, check=True, capture_output=True)
    out = {}
    for f in sorted(os.listdir(d)):
        if "gfx950" not in f:
            continue
        text = subprocess.run([LLVM + "llvm-readelf", "--notes", f], cwd=d, check=True, capture_output=True, text=True).stdout
        for k in re.split(r"\n\s*- \.a", text)[1:]:  # a kernel's entries begin with .agpr_count or .args
            name = re.search(r"\.name:\s+(\S*kernel\S*)", k)
            if name:
                out[name.group(1)] = {x: int(re.search(r"\.%s:\s+(\d+)" % x, k).group(1)) for x in ("vgpr_count", "vgpr_spill_count")}
    return out


def test_no_vector_spills(kernels):
    assert sum("attn_" in k for k in kernels) >= 22
    assert {k: v for k, v in kernels.items() if v["vgpr_spill_count"]} == {}


@pytest.mark.parametrize("heads", [5, 6, 7, 8])
def test_four_waves_per_simd(kernels, heads):
    mine = [v for k, v in kernels.items() if "attn_tiles_kernelILi64ELi%dE" % heads in k and "ELb1E" in k]
    assert len(mine) == 1 and mine[0]["vgpr_count"] <= 128


@pytest.mark.gpu
@pytest.mark.parametrize("group,splits", [(g, s + more) for g, s in ((5, 5), (6, 4), (7, 4), (8, 3)) for more in (0, 1)])
def test_merges_match(group, splits):
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    wl = workloads.make_workload("registers", 7, hq=2 * group, hkv=2, d=64, prefills=[],
                                 decodes=[(64, 700), (3, 450), (0, 17), (100, 1000), (600, 64 * splits + 600), (33, 640)])
    p, t, out, lse = run(wl, torch.device("cuda:0"), force_splits=splits, num_cus=8)
    assert p.info.decode_q_waves == group and p.info.num_decode_tiles > 0 and p.info.max_splits == splits
    assert p.launches()[2] == (splits > 28 // group)
    check_full(wl, out, lse)
    check_cache(wl, t)
