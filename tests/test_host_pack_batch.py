"""The pack kernel that takes its tensors in the kernel arguments, run from its source on the CPU (tests/emu) and compared
with the tile-table path and a plain concatenation; AddressSanitizer checks every address it forms."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = "/opt/rocm/lib/llvm/bin/clang++"


def _build(tmp_path_factory, pages):
    if not os.path.exists(CLANG):
        pytest.skip("ROCm clang not present")
    exe = str(tmp_path_factory.mktemp("emu") / "emu_pack_batch")
    subprocess.run([CLANG, "-x", "c++", "-std=c++17", "-O1", "-g", "-fsanitize=address", "-fno-omit-frame-pointer", "-DDSLLM_PACK_BATCH_PAGES=%du" % pages,
                    "-I", os.path.join(ROOT, "tests", "emu"), "-o", exe, os.path.join(ROOT, "tests", "emu", "emu_pack_batch.cpp")],
                   check=True, cwd=os.path.join(ROOT, "tests", "emu"))
    return exe


@pytest.fixture(scope="module")
def emu(tmp_path_factory):
    return {pages: _build(tmp_path_factory, pages) for pages in (64, 4000)}


# one tensor; batches that end by their pages (in the middle of a tensor, and exactly at one's end) and by their pieces
@pytest.mark.parametrize("pages,seed,n,limit,pieces_end,pages_end", [
    (64, 1, 1, 20000, 0, 0), (64, 2, 16, 3, 0, 0), (64, 3, 64, 4096, 0, 1), (64, 6, 40, 600000, 0, 23), (64, 7, 400, 30000, 0, 19),
    (4000, 8, 320, 3, 1, 0), (4000, 8, 321, 3, 1, 0), (4000, 8, 700, 4096, 2, 0)])
def test_batch_image_equals_the_table_path(emu, pages, seed, n, limit, pieces_end, pages_end):
    r = subprocess.run([emu[pages], str(seed), str(n), str(limit)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "full_pieces %d full_pages %d" % (pieces_end, pages_end) in r.stdout, r.stdout[-2000:] + r.stderr[-4000:]
