"""What ckpt_pack_image and ckpt_pack_image_noalloc ask the runtime about a list, what they refuse, and the image, on the CPU
model of the runtime (tests/emu/emu_pack_image.cpp) under AddressSanitizer."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = "/opt/rocm/lib/llvm/bin/clang++"
SOURCES = ("engine.cpp", "submit.cpp", "io_threads.cpp", "restore.cpp", "second_tier.cpp", "plan.cpp", "pack_kernels.hip", "pack_image.hip",
           "derive_kernels.hip")


def test_queries_refusals_and_image(tmp_path):
    if not os.path.exists(CLANG):
        pytest.skip("ROCm clang not present")
    exe = str(tmp_path / "emu_pack_image")
    subprocess.run([CLANG, "-x", "c++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-omit-frame-pointer", "-pthread",
                    "-I", os.path.join(ROOT, "tests", "emu"), "-o", exe, os.path.join(ROOT, "tests", "emu", "emu_pack_image.cpp"),
                    *[os.path.join(ROOT, "paper_2406_10707_amd", "csrc", f) for f in SOURCES]], check=True, cwd=os.path.join(ROOT, "tests", "emu"))
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    out = r.stdout + r.stderr
    assert r.returncode == 0 and out.strip() == "ok pack image", out[-6000:]
