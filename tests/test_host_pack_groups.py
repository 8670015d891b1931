"""The pack kernel's look-up by groups of pages, run from its source on the CPU with every launch allowed to make them and
in both block orders, and compared like the look-up without: with the tile-table path and a plain concatenation."""
import os
import subprocess

import pytest

from tests.test_host_pack_batch import CLANG, ROOT


@pytest.fixture(scope="module")
def emu(tmp_path_factory):
    if not os.path.exists(CLANG):
        pytest.skip("ROCm clang not present")
    exes = {}
    for runs_from in (1, 1 << 30):
        exes[runs_from] = str(tmp_path_factory.mktemp("emu") / ("emu_pack_groups_%d" % runs_from))
        subprocess.run([CLANG, "-x", "c++", "-std=c++17", "-O1", "-g", "-fsanitize=address", "-fno-omit-frame-pointer", "-DDSLLM_PACK_BATCH_PAGES=900u",
                        "-DDSLLM_PACK_GROUPS_FROM=1", "-DDSLLM_PACK_RUNS_FROM=%d" % runs_from, "-I", os.path.join(ROOT, "tests", "emu"), "-o", exes[runs_from],
                        os.path.join(ROOT, "tests", "emu", "emu_pack_batch.cpp")], check=True, cwd=os.path.join(ROOT, "tests", "emu"))
    return exes


# lists of the three sizes of the arguments; one page a piece (up to 32 groups of one page, more), pieces of many groups, groups of many pieces
@pytest.mark.parametrize("runs_from", [1, 1 << 30])
@pytest.mark.parametrize("seed,n,limit", [(1, 1, 3), (2, 1, 3000000), (3, 32, 3), (4, 33, 3), (5, 32, 400000), (6, 128, 4096), (7, 129, 4096), (8, 320, 3), (9, 330, 20000)])
def test_image_by_groups(emu, runs_from, seed, n, limit):
    r = subprocess.run([emu[runs_from], str(seed), str(n), str(limit)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout[-2000:] + r.stderr[-4000:]
