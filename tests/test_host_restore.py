"""Restores that the caller's stream reaches late (tests/emu/emu_restore.cpp), on the CPU model of streams and events, under
ThreadSanitizer and AddressSanitizer."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = "/opt/rocm/lib/llvm/bin/clang++"
SOURCES = ("engine.cpp", "submit.cpp", "io_threads.cpp", "restore.cpp", "second_tier.cpp", "plan.cpp", "pack_kernels.hip", "pack_image.hip",
           "derive_kernels.hip")


# chunks sent in pieces and scattered one by one, and sent whole and scattered together, two at a time and all of a super-chunk
@pytest.fixture(scope="module", params=[("thread", 1), ("thread", 128 << 10), ("address,undefined", 1), ("address,undefined", 8 << 20)])
def emu(request, tmp_path_factory):
    if not os.path.exists(CLANG):
        pytest.skip("ROCm clang not present")
    exe = str(tmp_path_factory.mktemp("emu") / "emu_restore")
    subprocess.run([CLANG, "-x", "c++", "-std=c++17", "-O1", "-g", "-fsanitize=" + request.param[0], "-fno-omit-frame-pointer", "-pthread",
                    "-DDSLLM_SCATTER_BYTES=%dull" % request.param[1], "-I", os.path.join(ROOT, "tests", "emu"), "-o", exe, os.path.join(ROOT, "tests", "emu", "emu_restore.cpp"),
                    *[os.path.join(ROOT, "paper_2406_10707_amd", "csrc", f) for f in SOURCES]], check=True, cwd=os.path.join(ROOT, "tests", "emu"))
    return exe


@pytest.mark.parametrize("reduce,direct_min", [(0, 0), (1, 0), (0, 100000), (1, 100000)])
def test_work_between_two_restores_reads_the_first_file(emu, tmp_path, reduce, direct_min):
    r = subprocess.run([emu, str(tmp_path), "order", str(reduce), str(direct_min)], capture_output=True, text=True, timeout=300)
    out = r.stdout + r.stderr
    assert r.returncode == 0 and out.strip() == "ok order", out[-6000:]


@pytest.mark.parametrize("reduce,direct_min", [(0, 0), (1, 0), (0, 100000)])
def test_a_failed_restore_writes_nothing_after_it_has_returned(emu, tmp_path, reduce, direct_min):
    r = subprocess.run([emu, str(tmp_path), "failed", str(reduce), str(direct_min)], capture_output=True, text=True, timeout=300)
    out = r.stdout + r.stderr
    assert r.returncode == 0 and out.strip() == "ok failed", out[-6000:]
