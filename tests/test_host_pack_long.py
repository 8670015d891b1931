"""The pack kernel with the arguments of a long list (1280 pieces, 128 groups of pages), run from its source on the CPU in both block
orders and compared like the short one: with the tile-table path and a plain concatenation."""
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
        exes[runs_from] = str(tmp_path_factory.mktemp("emu") / ("emu_pack_long_%d" % runs_from))
        subprocess.run([CLANG, "-x", "c++", "-std=c++17", "-O1", "-g", "-fsanitize=address", "-fno-omit-frame-pointer", "-DDSLLM_PACK_BATCH_PAGES=6000u",
                        "-DDSLLM_PACK_GROUPS_FROM=1", "-DDSLLM_PACK_RUNS_FROM=%d" % runs_from, "-DEMU_BATCH=LongPackBatch", "-DEMU_PIECES=kLongPackBatch",
                        "-I", os.path.join(ROOT, "tests", "emu"), "-o", exes[runs_from], os.path.join(ROOT, "tests", "emu", "emu_pack_batch.cpp")],
                       check=True, cwd=os.path.join(ROOT, "tests", "emu"))
    return exes


# the last batch with the arguments of each of the four sizes; batches that end by their pieces and by their pages
@pytest.mark.parametrize("runs_from", [1, 1 << 30])
@pytest.mark.parametrize("seed,n,limit,pieces_end,pages_end", [(1, 321, 3, 0, 0), (2, 1279, 3, 0, 0), (3, 1280, 4096, 1, 0), (4, 1281, 3, 1, 0), (5, 1313, 3, 1, 0),
                                                                (6, 1409, 3, 1, 0), (7, 1601, 3, 1, 0), (8, 2600, 3, 2, 0), (9, 400, 900000, 0, 3)])
def test_long_image_equals_the_table_path(emu, runs_from, seed, n, limit, pieces_end, pages_end):
    r = subprocess.run([emu[runs_from], str(seed), str(n), str(limit)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "full_pieces %d full_pages %d" % (pieces_end, pages_end) in r.stdout, r.stdout[-2000:] + r.stderr[-4000:]
