"""The hand-ordered GEMM forms, as compiled with the library's own flags: those whose matrix instructions are inline
assembly set every accumulator before the fence and write no operand right before its use, and no form spills."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2406_10707_amd import build
from tests.test_host_gemm_fence import HIPCC, _registers


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    if not shutil.which(HIPCC):
        pytest.skip("hipcc not present")
    out = str(tmp_path_factory.mktemp("isa") / "proxy.s")
    subprocess.run([HIPCC, "-x", "hip", "-S", "--cuda-device-only", os.path.join(build.CSRC, "proxy_kernels.hip"), "-o", out] + build.HIPCC_FLAGS,
                   check=True, capture_output=True)
    with open(out) as f:
        return f.read()


def test_inline_matrix_instructions_keep_their_distances(assembly):
    checked = 0
    for body in re.findall(r"^\w*gemm_bf16_tile_kernel\w*:.*?^\s*s_endpgm", assembly, re.S | re.M):
        lines = [line.split(";")[0].strip() if not line.strip().startswith(";") else line.strip() for line in body.splitlines()]
        if not any(x.startswith(";APP") or x.startswith(";;#ASMSTART") for x in lines) or "s_nop 7" not in lines:
            continue       # matrix instructions of the compiler's own
        checked += 1
        code = [x for x in lines if x and not x.startswith((".", ";"))]
        first = next(i for i, x in enumerate(code) if x.startswith("v_mfma"))
        accumulators = set().union(*[_registers(re.split(r"[\s,]+(?![^\[]*\])", x)[1]) for x in code if x.startswith("v_mfma")])
        written = {r for x in code[:first] if re.match(r"v_accvgpr_(write|mov)", x) for r in _registers(re.split(r"[\s,]+", x)[1])}
        fence = max(i for i, x in enumerate(code[:first]) if x == "s_nop 7")
        assert accumulators and accumulators <= written
        assert not any(re.match(r"v_accvgpr_(write|mov)", x) for x in code[fence:first])
        recent = []
        for x in code:
            op, _, rest = x.partition(" ")
            args = [a.strip() for a in re.split(r",\s*(?![^\[]*\])", rest)]
            if op.startswith("v_mfma"):
                assert not set().union(*recent) & set().union(*[_registers(a) for a in args]), x
            recent = (recent + [_registers(args[0]) if op.startswith("v_") and not op.startswith("v_mfma") else set()])[-2:]
    assert checked >= 6        # three forms, with 32-bit and with 64-bit addresses


def test_no_form_spills(assembly):
    spills = [int(n) for name, n in re.findall(r"\.name:\s+(\w*gemm_bf16\w*)\s.*?\.vgpr_spill_count:\s+(\d+)", assembly, re.S)]
    assert len(spills) >= 2 * 16 and not any(spills)
