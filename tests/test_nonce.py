"""The numbers that mark split partials as written (nonce.h): none twice, in a
process or across two, with an entropy source or without one, and no exception
leaves them. CPU only."""
import os
import re
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2607_04206_amd", "csrc")


@pytest.mark.parametrize("flags", [[], ["-DNO_ENTROPY"]])
def test_never_twice(tmp_path, flags):
    if not shutil.which("g++"):
        pytest.skip("needs g++")
    exe = str(tmp_path / "driver")
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", *flags, os.path.join(HERE, "sanitize", "nonce_driver.cpp"), "-o", exe], check=True)
    got = [int(x, 16) for _ in range(2) for x in subprocess.run([exe], capture_output=True, text=True, check=True).stdout.split()]
    assert len(got) == 2000 == len(set(got)) and 0 not in got


def test_the_forward_takes_them_from_there():
    with open(os.path.join(CSRC, "attn_fwd.hip")) as f:
        text = f.read()
    assert '#include "nonce.h"' in text and not re.search(r"random_device|uint64_t next_nonce", text)
