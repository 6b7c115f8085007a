"""The numbering that deals workgroups with work in the last wave to all XCDs (tests/host/numbering.cpp).  CPU only."""
import os
import shutil
import subprocess

import pytest

import paper_2408_11417_amd as sk
from tests.test_gpu_gemm import SPREAD

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2408_11417_amd", "csrc")
DP, SK, BF16, E4M3 = sk.SK_POLICY_DP, sk.SK_POLICY_ALL_SK, sk.SK_BF16, sk.SK_FP8_E4M3


@pytest.fixture(scope="module")
def numbering(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    exe = str(tmp_path_factory.mktemp("numbering") / "numbering")
    res = subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                          os.path.join(ROOT, "tests", "host", "numbering.cpp"), os.path.join(CSRC, "streamk_plan.cpp"), "-o", exe],
                         stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert res.returncode == 0, res.stdout

    def run(*args):
        res = subprocess.run([exe] + [str(a) for a in args], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
        assert res.returncode == 0, res.stdout
        return res.stdout.strip()
    return run


def test_spread_ids_are_a_permutation(numbering):
    assert numbering("bijection") == "ok"


@pytest.mark.parametrize("shape,blk,grid,policy,dealt", SPREAD)
def test_plans_that_run_the_spread_numbering_on_the_gpu_do_so(numbering, shape, blk, grid, policy, dealt):
    assert int(numbering(*shape, policy, *blk, grid, BF16)) == dealt


@pytest.mark.parametrize("shape,blk,policy,dtype,dealt", [
    # a last wave of few tiles behind a full one stays together, a larger one is dealt
    ((128 * 12, 128 * 22, 576), (128, 128, 64), DP, BF16, 0), ((128 * 15, 128 * 20, 576), (128, 128, 64), DP, BF16, 0), ((128 * 19, 128 * 20, 576), (128, 128, 64), DP, BF16, 124),
    ((256 * 12, 128 * 22, 576), (256, 128, 64), DP, BF16, 0), ((256 * 15, 128 * 20, 576), (256, 128, 64), DP, BF16, 44), ((128 * 14, 256 * 20, 1152), (128, 256, 128), DP, E4M3, 0),
    ((256 * 20, 256 * 26, 576), (256, 256, 64), DP, BF16, 0), ((256 * 19, 256 * 30, 576), (256, 256, 64), DP, BF16, 58), ((256 * 19, 256 * 30, 320), (256, 256, 64), DP, BF16, 0), ((256 * 20, 256 * 26, 2304), (256, 256, 64), DP, BF16, 0),
    ((256 * 20, 256 * 33, 2304), (256, 256, 64), DP, BF16, 148),
    # less than one wave
    ((256 * 11, 256 * 20, 576), (256, 256, 64), DP, BF16, 220), ((64 * 115, 128 * 2, 576), (64, 128, 64), DP, BF16, 230), ((256 * 15, 256 * 17, 576), (256, 256, 64), DP, BF16, 0),
    ((32 * 8, 128 * 8, 1024), (32, 128, 64), DP, BF16, 64), ((32 * 8, 128 * 8, 960), (32, 128, 64), DP, BF16, 0), ((256 * 3, 256 * 5, 576), (256, 256, 64), DP, BF16, 0),
    # Stream-K plans with empty ranges: by how many workgroups are busy
    ((70, 119, 4092), (16, 128, 64), SK, BF16, 160), ((112, 256, 896), (16, 128, 64), SK, BF16, 196), ((16, 128, 1984), (16, 128, 64), SK, BF16, 0)])
def test_where_the_numbering_is_spread(numbering, shape, blk, policy, dtype, dealt):
    assert int(numbering(*shape, policy, *blk, 256, dtype)) == dealt
