"""Block order of the launch that holds prefill-shaped tiles and block decodes
(mixed_order.h), listed on the CPU: it ends for every mix, holds each tile
exactly once and hardly an empty block."""
import os
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def order(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("needs g++")
    exe = str(tmp_path_factory.mktemp("order") / "driver")
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", os.path.join(HERE, "sanitize", "mixed_order_driver.cpp"), "-o", exe], check=True)

    def list_blocks(mixes):
        r = subprocess.run([exe], input="\n".join("%d %d %d" % m for m in mixes), capture_output=True, text=True, timeout=120, check=True)
        return [tuple(int(x) for x in line.split()) for line in r.stdout.splitlines()]
    return list_blocks


# few decode groups beside very many prefill blocks (one in 65,536 and fewer) and the reverse
EXTREME = [(524536, 257, 256), (524537, 257, 256), (524544, 264, 256), (2100000, 33 * 8, 256), (1 << 22, 300, 256), (1049132 - 257, 257, 256),
           (257, 1 << 22, 256), (1 << 22, 1 << 22, 256), (3, 1 << 21, 16)]


def mixes():
    rng = np.random.default_rng(0)
    out = [(p, d, r) for p in (1, 7, 8, 9, 255, 256, 257, 264, 513) for d in (1, 8, 255, 256, 257, 263, 265, 600) for r in (16, 256)]
    for _ in range(300):
        out.append((int(np.exp(rng.uniform(0, 11))), int(np.exp(rng.uniform(0, 11))), int(rng.choice([16, 256, 1 << 20]))))
    return out + EXTREME


def test_every_tile_once(order):
    lines = order(mixes())
    assert len(lines) == len(mixes())
    for mix, (blocks, empty, bad, *_) in zip(mixes(), lines):
        assert bad == 0, mix
        assert blocks - empty == mix[0] + mix[1] and empty <= 62, mix
