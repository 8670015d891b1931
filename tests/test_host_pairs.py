"""The kernels that check and regenerate derived tensors, run from their source on the CPU (tests/emu) over tables of large and
small work items, in one launch and in several; AddressSanitizer checks every address they form."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = "/opt/rocm/lib/llvm/bin/clang++"


@pytest.fixture(scope="module", params=[1 << 22, 5])
def emu(request, tmp_path_factory):
    if not os.path.exists(CLANG):
        pytest.skip("ROCm clang not present")
    exe = str(tmp_path_factory.mktemp("emu") / "emu_pairs")
    subprocess.run([CLANG, "-x", "c++", "-std=c++17", "-O1", "-g", "-fsanitize=address", "-fno-omit-frame-pointer", "-DDSLLM_PAIR_TILES_PER_LAUNCH=%du" % request.param,
                    "-I", os.path.join(ROOT, "tests", "emu"), "-o", exe, os.path.join(ROOT, "tests", "emu", "emu_pairs.cpp"),
                    os.path.join(ROOT, "paper_2406_10707_amd", "csrc", "plan.cpp")], check=True, cwd=os.path.join(ROOT, "tests", "emu"))
    return exe


# small items only (a number that four does not divide among them), one pair, all sizes
@pytest.mark.parametrize("seed,n,limit", [(1, 1, 3), (2, 1, 20000), (3, 37, 512), (4, 7, 300), (5, 60, 10000), (6, 60, 30000)])
def test_check_and_regeneration(emu, seed, n, limit):
    r = subprocess.run([emu, str(seed), str(n), str(limit)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.startswith("ok items"), r.stdout[-2000:] + r.stderr[-4000:]
