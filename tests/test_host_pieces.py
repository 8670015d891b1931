"""The engine's source on the CPU model of streams and events (tests/emu), built so that a chunk goes to and from the file in
several pieces and a snapshot's first chunk is packed apart: the scenarios of the engine's own test, under ThreadSanitizer and under AddressSanitizer."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = "/opt/rocm/lib/llvm/bin/clang++"
SOURCES = ("engine.cpp", "submit.cpp", "io_threads.cpp", "restore.cpp", "second_tier.cpp", "plan.cpp", "pack_kernels.hip", "pack_image.hip",
           "derive_kernels.hip")


@pytest.mark.parametrize("sanitizer,piece", [("thread", 8192), ("thread", 12288), ("address,undefined", 4096)])
def test_engine_scenarios_with_chunks_in_several_pieces(tmp_path, sanitizer, piece):
    if not os.path.exists(CLANG):
        pytest.skip("ROCm clang not present")
    exe = str(tmp_path / "emu_engine")
    subprocess.run([CLANG, "-x", "c++", "-std=c++17", "-O1", "-g", "-fsanitize=" + sanitizer, "-fno-omit-frame-pointer", "-pthread",
                    "-DDSLLM_PIECE_BYTES=%dull" % piece, "-DDSLLM_HEAD_APART_TILES=1", "-DDSLLM_SCATTER_BYTES=%dull" % (1 if piece == 8192 else 128 << 10), "-I", os.path.join(ROOT, "tests", "emu"), "-o", exe, os.path.join(ROOT, "tests", "emu", "emu_engine.cpp"),
                    *[os.path.join(ROOT, "paper_2406_10707_amd", "csrc", f) for f in SOURCES]], check=True, cwd=os.path.join(ROOT, "tests", "emu"))
    work = tmp_path / "files"
    work.mkdir()
    r = subprocess.run([exe, str(work), "5"], capture_output=True, text=True, timeout=600)
    out = r.stdout + r.stderr
    assert r.returncode == 0 and "FAILED" not in out and "Sanitizer" not in out and "runtime error" not in out, out[-6000:]
    assert out.count("ok policy") == 12 and out.count("snapshots copied") == 3
    r = subprocess.run([exe, "--failed-chunk", str(work)], capture_output=True, text=True, timeout=300)
    out = r.stdout + r.stderr
    assert r.returncode == 0 and "FAILED" not in out and "Sanitizer" not in out and out.count("ok failed chunk") == 2, out[-6000:]
