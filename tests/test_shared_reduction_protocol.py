"""The shared reduction with any number of workgroups on the device at once (tests/host/shared_reduction.cpp).  CPU only."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2408_11417_amd", "csrc")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    exe = str(tmp_path_factory.mktemp("shared") / "shared_reduction")
    res = subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-pthread", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                          os.path.join(ROOT, "tests", "host", "shared_reduction.cpp"), os.path.join(CSRC, "streamk_plan.cpp"), "-o", exe],
                         stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert res.returncode == 0, res.stdout
    return exe


# ranges that straddle tiles and that end with them, few and many workgroups per tile, more of them than units
@pytest.mark.parametrize("shape,blk,grid", [((224, 576, 27328), (64, 128, 64), 256), ((720, 896, 12272), (128, 128, 64), 256), ((256, 512, 16384), (64, 64, 128), 256),
                                            ((512, 6656, 2496), (256, 256, 64), 256), ((128, 448, 2304), (64, 64, 128), 256), ((256, 256, 20480), (256, 256, 64), 320)])
def test_the_launch_ends_with_every_unit_stored_once(driver, shape, blk, grid):
    for slots in (1, 8, 16, 20, 24, 28, 32, grid // 8):
        for polls, order in ((0, 1), (3, 0), (40, 1), (40, 2)):
            res = subprocess.run([driver] + [str(v) for v in shape + blk + (grid, slots, polls, order)], stdout=subprocess.PIPE,
                                 stderr=subprocess.STDOUT, text=True, timeout=120)
            assert res.returncode == 0 and res.stdout.startswith("ok "), (slots, polls, order, res.stdout)
            if slots == 1 and order == 1:          # one XCD's workgroups run one by one, and neighbours share a tile
                assert " 0 shares" not in res.stdout, (slots, polls, order, res.stdout)
