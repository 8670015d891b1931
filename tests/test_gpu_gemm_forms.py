"""Every form that the proxy's GEMM chooses among, with tiles that end at the edge of C and tiles that reach over it in
either direction, against the float64 product. K is as short as the form is chosen for, in steps that its stages in LDS
divide and do not divide."""
import numpy as np
import pytest

from oracle import proxy_oracle as po
from paper_2406_10707_amd import binding as B
from paper_2406_10707_amd import harness
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu

# by the form that they take (tests/test_host_gemm_forms.py asks the choice itself)
FORMS = {
    "256x256": [(2816, 5120, 256), (4736, 2944, 256), (2816, 5120, 1472)],
    "224x256": [(4480, 2816, 256), (3328, 3840, 256), (2816, 4480, 320)],
    "256x192": [(2048, 4992, 256), (3072, 3200, 320), (2176, 4736, 320)],
    "160x256": [(2560, 3328, 256), (4736, 1792, 320), (2432, 3456, 256)],
    "192x128 by 2": [(1152, 4224, 256), (2944, 1792, 320)],
    "160x128": [(2560, 1664, 256), (4736, 896, 320)],
    "128x128": [(4992, 640, 256), (640, 4992, 320)],
    "128x128 by 2": [(4480, 1408, 448)],
    "128x96": [(2816, 768, 256), (1664, 1280, 320)],
    "64x128 by 2": [(512, 2816, 320), (512, 2816, 448)],
    "96x64 by 2": [(768, 1408, 256), (640, 1664, 320)],
    "64x64 by 2": [(384, 768, 1408), (640, 1408, 1088)],
    "64x64 by 3": [(128, 128, 256), (256, 384, 320)],
    "32x64 K/4": [(256, 1536, 2048 + 64)],
    "32x32 K/4": [(384, 256, 2048 + 64), (128, 128, 1024), (512, 512, 1664), (128, 640, 1152), (128, 1664, 1472)],
    # the order left to the compiler, four waves a tile: a few steps of K, and up to K = 192 a single round of blocks or K = 64
    "128x128 compiled": [(4480, 1408, 256), (2176, 3200, 64), (3072, 2176, 192), (2048, 4096, 64)],
    # K up to 192; strips of 1 to 7 rows of tiles; the most tiles of 64 x 64
    "64x64 short": [(2304, 1152, 192), (1152, 1024, 192), (128, 128, 64), (384, 640, 64), (640, 1664, 128), (1408, 640, 192), (1920, 896, 64), (1024, 3072, 64)],
    "64x128 short": [(128, 25088, 128), (1664, 3584, 192), (3072, 4096, 64)],
    "128x128 short, eight waves": [(2944, 4736, 128), (3072, 4224, 192)],
}


@pytest.mark.parametrize("m,n,k", [shape for shapes in FORMS.values() for shape in shapes])
def test_gemm_form_against_float64(m, n, k):
    print(f"gemm {m}x{n}x{k}", flush=True)
    rng = np.random.default_rng(m + 3 * n + 7 * k)
    a = po.bf16_bits(rng.standard_normal((m, k)).astype(np.float32))
    b = po.bf16_bits(rng.standard_normal((n, k)).astype(np.float32))
    # rows behind the operands' last are there and are no numbers: whatever a tile over the edge reads is not stored
    nan = np.full((256, k), 0x7FC0, dtype=np.uint16)
    da, db, dc = harness.DevBuf(2 * (m + 256) * k), harness.DevBuf(2 * (n + 256) * k), harness.DevBuf(2 * m * n + 4096)
    da.upload(np.concatenate([a, nan]))
    db.upload(np.concatenate([b, nan]))
    ref, ref_abs = po.gemm_bf16(a, b)
    # f32 sums of K products in any order: K 2^-23 sum |a||b|; one rounding to bf16: 2^-8 |c|
    bound = k * 2.0 ** -23 * ref_abs + 2.0 ** -8 * np.abs(ref) + 1e-30
    first = None
    for _ in range(2):       # the same bits each time: nothing depends on the order in which waves arrive
        B.proxy_device_fill_async(dc.ptr, 0xEE, dc.nbytes, 0)
        B.proxy_gemm_bf16(da.ptr, db.ptr, dc.ptr, m, n, k, 0)
        harness.synchronize()
        out = gu.download(dc)
        assert np.all(out[2 * m * n:] == 0xEE)
        got = po.bf16_to_f64(out[:2 * m * n].view(np.uint16).reshape(m, n))
        assert np.all(np.abs(got - ref) <= bound), float(np.max(np.abs(got - ref) / bound))
        assert first is None or np.array_equal(first, out)
        first = out
    for x in (da, db, dc):
        x.free()
