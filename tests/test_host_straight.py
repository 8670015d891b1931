"""Small shards packed straight into the ring (tests/emu/emu_straight.cpp) under ThreadSanitizer and AddressSanitizer."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = "/opt/rocm/lib/llvm/bin/clang++"
SOURCES = ("engine.cpp", "submit.cpp", "io_threads.cpp", "restore.cpp", "second_tier.cpp", "plan.cpp", "pack_kernels.hip", "pack_image.hip",
           "derive_kernels.hip")


@pytest.mark.parametrize("sanitizer", ["thread", "address,undefined"])
def test_files_hold_the_state_at_their_boundary(tmp_path, sanitizer):
    if not os.path.exists(CLANG):
        pytest.skip("ROCm clang not present")
    exe = str(tmp_path / "emu_straight")
    subprocess.run([CLANG, "-x", "c++", "-std=c++17", "-O1", "-g", "-fsanitize=" + sanitizer, "-fno-omit-frame-pointer", "-pthread",
                    "-I", os.path.join(ROOT, "tests", "emu"), "-o", exe, os.path.join(ROOT, "tests", "emu", "emu_straight.cpp"),
                    *[os.path.join(ROOT, "paper_2406_10707_amd", "csrc", f) for f in SOURCES]], check=True, cwd=os.path.join(ROOT, "tests", "emu"))
    for policy in (0, 1):
        work = tmp_path / f"files{policy}"
        work.mkdir()
        r = subprocess.run([exe, str(work), str(policy)], capture_output=True, text=True, timeout=300)
        out = r.stdout + r.stderr
        assert r.returncode == 0 and out.strip() == f"ok straight policy {policy}", out[-6000:]
