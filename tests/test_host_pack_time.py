"""The pack time a snapshot reports (tests/emu/emu_pack_time.cpp) is the launches' own, without what passes between them."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = "/opt/rocm/lib/llvm/bin/clang++"
SOURCES = ("engine.cpp", "submit.cpp", "io_threads.cpp", "restore.cpp", "second_tier.cpp", "plan.cpp", "pack_kernels.hip", "pack_image.hip",
           "derive_kernels.hip")


def test_pack_time_is_that_of_the_launches(tmp_path):
    if not os.path.exists(CLANG):
        pytest.skip("ROCm clang not present")
    exe = str(tmp_path / "emu_pack_time")
    subprocess.run([CLANG, "-x", "c++", "-std=c++17", "-O1", "-g", "-fsanitize=thread", "-fno-omit-frame-pointer", "-pthread",
                    "-DDSLLM_HEAD_APART_TILES=1", "-I", os.path.join(ROOT, "tests", "emu"), "-o", exe, os.path.join(ROOT, "tests", "emu", "emu_pack_time.cpp"),
                    *[os.path.join(ROOT, "paper_2406_10707_amd", "csrc", f) for f in SOURCES]], check=True, cwd=os.path.join(ROOT, "tests", "emu"))
    r = subprocess.run([exe, str(tmp_path)], capture_output=True, text=True, timeout=300)
    out = r.stdout + r.stderr
    assert r.returncode == 0 and out.strip() == "ok pack time", out[-6000:]
