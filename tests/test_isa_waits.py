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
def text(tmp_path_factory):
    if not os.path.exists(OBJDUMP):
        pytest.skip("needs llvm-objdump")
    d = str(tmp_path_factory.mktemp("isa"))
    shutil.copy(_lib.LIB_PATH, d)
    subprocess.run([OBJDUMP, "--offloading", os.path.basename(_lib.LIB_PATH)], cwd=d, check=True, capture_output=True)
    lines = []
    for f in sorted(os.listdir(d)):
        if "gfx950" in f:
            lines += subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", f], cwd=d, check=True, capture_output=True, text=True).stdout.splitlines()
    assert any("attn_tiles_kernel" in x for x in lines)
    return lines


@pytest.fixture(scope="module")
def listing(text):
    return [x.split("//")[0].strip() for x in text]


@pytest.fixture(scope="module")
def kernels(text):
    """name -> [(address, operation, operands)] of the attention kernels"""
    out, code = {}, None
    for line in text:
        m = re.match(r"[0-9a-f]+ <(\S+)>:", line)
        if m:
            code = out.setdefault(m.group(1), []) if "attn" in m.group(1) else None
            continue
        m = re.match(r"\t(\S+)\s*(.*?)\s*// ([0-9A-F]+):", line)
        if m and code is not None:
            code.append((int(m.group(3), 16), m.group(1), m.group(2)))
    return out


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


# What the compiler itself keeps between a 32 x 32 x 16 MFMA and the first other access of its result.
MFMA_WAIT = 12


def registers(text):
    out = set()
    for m in re.finditer(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)", text):
        lo = int(m.group(2) or m.group(4))
        out |= {(m.group(1), i) for i in range(lo, int(m.group(3) or lo) + 1)}
    return out


def test_mfma_results_are_waited_for_on_every_path(kernels):
    """Branches are followed: a uniform branch between the last MFMA and the
    epilogue once held too few wait states on one of its paths."""
    checked = 0
    for name, code in kernels.items():
        at = {a: i for i, (a, _, _) in enumerate(code)}
        regs = [registers(args) for _, _, args in code]
        for i, (_, op, args) in enumerate(code):
            if not op.startswith("v_mfma"):
                continue
            checked += 1
            result = registers(args[:args.index("]") + 1])
            paths, best = [(i + 1, 0)], {}
            while paths:
                j, waited = paths.pop()
                while j < len(code) and waited < MFMA_WAIT and best.get(j, MFMA_WAIT) > waited:
                    best[j] = waited
                    addr, op2, args2 = code[j]
                    mfma = op2.startswith("v_mfma")  # (dependent ones are interlocked)
                    assert mfma or not regs[j] & result, (name, hex(code[i][0]), hex(addr), waited)
                    if (mfma and regs[j] & result) or op2 == "s_endpgm":
                        break
                    waited += states(op2 + " " + args2)
                    if op2 == "s_branch" or op2.startswith("s_cbranch"):
                        off = int(args2.split()[0])
                        paths.append((at[addr + 4 + 4 * (off - 65536 * (off > 32767))], waited))
                        if op2 == "s_branch":
                            break
                    j += 1
    assert checked > 500
