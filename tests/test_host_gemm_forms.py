"""Which form the proxy's GEMM takes, asked of the choice itself (csrc/gemm_forms.hpp): the shapes of the GPU tests take the
forms that they stand for, and there is one for every form."""
import os
import re
import subprocess

import pytest

from tests.test_gpu_gemm_forms import FORMS
from tests.test_gpu_gemm_shapes import WIDE_FORMS, WIDE_K

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def forms(tmp_path_factory):
    """forms(shapes) -> [(name, blocks, threads of a block)]"""
    exe = str(tmp_path_factory.mktemp("forms") / "gemm_form")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-o", exe, os.path.join(ROOT, "tests", "emu", "gemm_form.cpp")], check=True)

    def ask(shapes):
        out = subprocess.run([exe], input="".join("%d %d %d\n" % s for s in shapes), capture_output=True, text=True, check=True).stdout
        return [(name, int(blocks), int(threads)) for name, blocks, threads in (line.rsplit(",", 2) for line in out.splitlines())]

    return ask


@pytest.fixture(scope="module")
def table():
    """[(name, built for 64-bit addresses too)]"""
    with open(os.path.join(ROOT, "paper_2406_10707_amd", "csrc", "gemm_forms.hpp")) as f:
        return [(name, wide == "true") for name, wide in re.findall(r'^    \{"([^"]+)", \d+, \d+, \d+, \d, (true|false), ', f.read(), re.M)]


def test_every_form_has_shapes_that_take_it(forms, table):
    assert len(table) == 19 and [name for name, _ in table] == list(FORMS)
    for name, shapes in FORMS.items():
        assert shapes and [taken for taken, _, _ in forms(shapes)] == [name] * len(shapes)


def test_every_form_with_64_bit_addresses_has_a_shape_that_takes_it(forms, table):
    assert [name for name, wide in table if wide] == list(WIDE_FORMS)
    for name, shapes in WIDE_FORMS.items():
        assert shapes and [taken for taken, _, _ in forms([(m, n, WIDE_K) for m, n in shapes])] == [name] * len(shapes)


def test_only_forms_built_for_64_bit_addresses_are_taken_with_them(forms, table):
    sizes = [128, 256, 384, 640, 1024, 1408, 2048, 4480, 8192, 16384, 20608, 21760, 33280]
    shapes = [(m, n, k) for m in sizes for n in sizes for k in (WIDE_K, 1 << 26, (1 << 31) - 64)]
    assert {name for name, _, _ in forms(shapes)} <= {name for name, wide in table if wide}


@pytest.mark.parametrize("k", [64, 128, 192, 256, 320, 1024])
def test_a_grid_has_fewer_work_items_than_32_bits_count(forms, k):
    """Up to a C of 288 GB, square and flat."""
    shapes = []
    for rows in (128, 1 << 14, 1 << 16, 1 << 18, 128 * 2897):
        for elements in (1 << 35, 1 << 36, (1 << 37) - (1 << 30), 1 << 37, 144 * 10 ** 9):
            cols = -(-elements // rows // 128) * 128
            if cols < 1 << 31:
                shapes.append((rows, cols, k))
    assert len(shapes) >= 20
    for shape, (name, blocks, threads) in zip(shapes, forms(shapes)):
        assert blocks * threads < 1 << 32, (shape, name)
