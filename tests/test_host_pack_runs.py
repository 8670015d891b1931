"""The pack kernel's other block order (for tensors off the 128-byte lines), run from its source on the CPU with every
launch allowed to take it, and compared like the first one: with the tile-table path and a plain concatenation."""
import os
import subprocess

import pytest

from tests.test_host_pack_batch import CLANG, ROOT


@pytest.fixture(scope="module")
def emu(tmp_path_factory):
    if not os.path.exists(CLANG):
        pytest.skip("ROCm clang not present")
    exe = str(tmp_path_factory.mktemp("emu") / "emu_pack_runs")
    subprocess.run([CLANG, "-x", "c++", "-std=c++17", "-O1", "-g", "-fsanitize=address", "-fno-omit-frame-pointer", "-DDSLLM_PACK_BATCH_PAGES=64u",
                    "-DDSLLM_PACK_RUNS_FROM=1", "-I", os.path.join(ROOT, "tests", "emu"), "-o", exe, os.path.join(ROOT, "tests", "emu", "emu_pack_batch.cpp")],
                   check=True, cwd=os.path.join(ROOT, "tests", "emu"))
    return exe


# one page; batches of pages that 16 divides and does not divide (64 blocks are four times 16 pages), ended by pages or by the list
@pytest.mark.parametrize("seed,n,limit", [(2, 1, 3), (2, 16, 3), (3, 64, 4096), (6, 40, 600000), (7, 400, 30000)])
def test_image_in_runs(emu, seed, n, limit):
    r = subprocess.run([emu, str(seed), str(n), str(limit)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout[-2000:] + r.stderr[-4000:]
