"""Snapshots in parts and restores of files larger than the ring (tests/emu/emu_parts.cpp), on the CPU model of streams and events,
under ThreadSanitizer and AddressSanitizer."""
import os
import subprocess

import pytest

from tests.test_host_restore import CLANG, ROOT, SOURCES


def _build(tmp_path_factory, sanitizer, *sizes):
    if not os.path.exists(CLANG):
        pytest.skip("ROCm clang not present")
    exe = str(tmp_path_factory.mktemp("emu") / "emu_parts")
    subprocess.run([CLANG, "-x", "c++", "-std=c++17", "-O1", "-g", "-fsanitize=" + sanitizer, "-fno-omit-frame-pointer", "-pthread", *sizes, "-I", os.path.join(ROOT, "tests", "emu"), "-o", exe,
                    os.path.join(ROOT, "tests", "emu", "emu_parts.cpp"), *[os.path.join(ROOT, "paper_2406_10707_amd", "csrc", f) for f in SOURCES]],
                   check=True, cwd=os.path.join(ROOT, "tests", "emu"))
    return exe


@pytest.fixture(scope="module", params=["thread", "address,undefined"])
def emu(request, tmp_path_factory):
    return _build(tmp_path_factory, request.param, "-DDSLLM_PIECE_BYTES=4096ull", "-DDSLLM_SCATTER_BYTES=1ull")


def _run(emu, *args):
    r = subprocess.run([emu, *map(str, args)], capture_output=True, text=True, timeout=300)
    out = r.stdout + r.stderr
    assert r.returncode == 0 and out.strip() == "ok " + args[1], out[-6000:]


def test_the_end_of_the_copies_is_seen_before_the_last_chunk_is_written(emu, tmp_path):
    _run(emu, tmp_path, "end")


def test_a_straight_snapshot_does_not_wait_for_the_next_one(emu, tmp_path):
    _run(emu, tmp_path, "straight")


def test_a_last_piece_does_not_wait_for_the_next_snapshot(tmp_path_factory, tmp_path):
    _run(_build(tmp_path_factory, "thread", "-DDSLLM_PIECE_BYTES=8192ull", "-DDSLLM_HEAD_APART_TILES=1000000"), tmp_path, "late")


# chunks sent in pieces, and (more than sixteen pieces) as a whole in between
@pytest.mark.parametrize("chunk,slots", [(64 << 10, 2), (64 << 10, 3), (128 << 10, 2), (128 << 10, 3), (128 << 10, 20)])
def test_a_restore_keeps_two_chunks_under_way(emu, tmp_path, chunk, slots):
    _run(emu, tmp_path, "restore", chunk, slots)


def test_a_context_has_the_events_that_it_uses(tmp_path_factory, tmp_path):
    _run(_build(tmp_path_factory, "address,undefined"), tmp_path, "events")


# pieces whose quarters are whole pages and pieces whose quarters are not, chunks of fewer and of more pages than four times the parts
@pytest.mark.parametrize("piece", [4096, 8192, 12288, 16384])
def test_no_piece_is_written_before_it_has_landed(tmp_path_factory, tmp_path, piece):
    emu = _build(tmp_path_factory, "thread", "-DDSLLM_PIECE_BYTES=%dull" % piece)
    for chunk in (64 << 10, 256 << 10, 416 << 10):
        _run(emu, tmp_path, "one", chunk)
