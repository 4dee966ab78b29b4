"""Wait states in the instructions of the built library. Those that the compiler
does not put into inline assembly: an SGPR written by the VALU (a spilled base
comes back by v_readlane) is read by a memory instruction at the earliest five
wait states later, and the data registers of a 16-byte store are written again
at the earliest two after it; the assembly blocks hold them themselves, whatever
the compiler puts around them. And those between an MFMA and the use of its
result. CPU only."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2607_04206_amd import _lib

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.fixture(scope="module")
def listing(tmp_path_factory):
    if not os.path.exists(OBJDUMP):
        pytest.skip("needs llvm-objdump")
    d = str(tmp_path_factory.mktemp("isa"))
    shutil.copy(_lib.LIB_PATH, d)
    subprocess.run([OBJDUMP, "--offloading", os.path.basename(_lib.LIB_PATH)], cwd=d, check=True, capture_output=True)
    lines = []
    for f in sorted(os.listdir(d)):
        if "gfx950" in f:
            out = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", f], cwd=d, check=True, capture_output=True, text=True).stdout
            lines += [x.split("//")[0].strip() for x in out.splitlines()]
    assert any("attn_tiles_kernel" in x for x in lines)
    return lines


def states(ins):
    m = re.match(r"s_nop (\d+)", ins)
    return int(m.group(1)) + 1 if m else 1


def test_page_copies_hold_five_wait_states(listing):
    starts = [i for i, x in enumerate(listing) if re.match(r"s_mov_b32 s\d+, m0$", x)]
    assert len(starts) > 100
    from_sgprs = 0
    for i in starts:
        waited = 0
        for j in range(i, i + 8):
            if listing[j].startswith("global_load_lds_dwordx4"):
                break
            assert re.match(r"s_(mov_b32|nop)", listing[j]), listing[i:j + 1]
            waited += states(listing[j])
        if re.search(r", s\[\d+:\d+\]", listing[j]):
            from_sgprs += 1
            assert waited >= 5, listing[i:j + 1]
        else:
            assert listing[j].startswith("global_load_lds_dwordx4") and ", off" in listing[j], listing[i:j + 1]
    assert from_sgprs > 50


def test_partial_stores_hold_two_wait_states(listing):
    stores = [i for i, x in enumerate(listing) if x.startswith("global_store_dwordx4") and x.endswith("sc1")]
    assert len(stores) > 50
    for i in stores:
        assert re.match(r"s_nop [1-9]", listing[i + 1]), listing[i:i + 2]
