"""The large GEMM kernel's matrix instructions are inline assembly, for which the compiler inserts no wait states: an operand
that an ordinary vector instruction has written needs two of them before a matrix instruction reads it. Read from the
assembly that the kernel's source compiles to with the library's own flags."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2406_10707_amd import build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def kernel(tmp_path_factory):
    if not shutil.which(HIPCC):
        pytest.skip("hipcc not present")
    out = str(tmp_path_factory.mktemp("isa") / "proxy.s")
    subprocess.run([HIPCC, "-x", "hip", "-S", "--cuda-device-only", os.path.join(build.CSRC, "proxy_kernels.hip"), "-o", out] + build.HIPCC_FLAGS,
                   check=True, capture_output=True)
    with open(out) as f:
        text = f.read()
    found = re.findall(r"^\w*gemm_bf16_256_kernel\w*:.*?^\s*s_endpgm", text, re.S | re.M)
    assert found
    return [[line.split(";")[0].strip() for line in body.splitlines()] for body in found]


def _registers(operand):
    m = re.fullmatch(r"([av])(?:(\d+)|\[(\d+):(\d+)\])", operand)
    if not m:
        return set()
    lo, hi = (int(m[2]), int(m[2])) if m[2] else (int(m[3]), int(m[4]))
    return {m[1] + str(r) for r in range(lo, hi + 1)}


def test_accumulators_are_set_before_the_fence(kernel):
    for body in kernel:
        first = next(i for i, line in enumerate(body) if line.startswith("v_mfma"))
        writes = [i for i, line in enumerate(body[:first]) if re.match(r"v_accvgpr_(write|mov)", line)]
        fences = [i for i, line in enumerate(body[:first]) if line == "s_nop 7"]
        assert len(writes) >= 256 and fences and fences[-1] > writes[-1], (writes[-1], fences, first)


def test_no_operand_is_written_right_before_its_use(kernel):
    for body in kernel:
        seen = 0
        recent = []      # registers written by the latest two instructions (the loop's jump back counts as none)
        for line in [x for x in body if x and not x.startswith(".")]:
            op, _, rest = line.partition(" ")
            args = [a.strip() for a in re.split(r",\s*(?![^\[]*\])", rest)]
            if op.startswith("v_mfma"):
                seen += 1
                assert not set().union(*recent) & set().union(*[_registers(a) for a in args]), line
            recent = (recent + [_registers(args[0]) if op.startswith("v_") and not op.startswith("v_mfma") else set()])[-2:]
        assert seen >= 128
