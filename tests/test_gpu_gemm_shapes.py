"""The proxy's GEMM over its range (the fewest steps of K, an odd number of them, steps that only some groups of waves have, an
odd number of tiles, a long K, many tiles of a flat C), against the float64 product. Every form that it chooses among:
test_gpu_gemm_forms.py."""
import numpy as np
import pytest

from oracle import proxy_oracle as po
from paper_2406_10707_amd import binding as B
from paper_2406_10707_amd import harness
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu

SHAPES = [(3072, 4096, 256), (3072, 4096, 320), (4096, 3328, 448),       # about 200 and more of the largest tiles
          (2176, 2048, 64), (2176, 2048, 192), (128, 67328, 128),        # more 64 x 64 tiles than are under way at once, short K
          (1536, 2048, 64), (1664, 1920, 320), (2432, 3456, 16384),
          (1152, 1024, 64), (1024, 1152, 576), (128, 128, 64), (256, 128, 448),     # fewer tiles
          (640, 1280, 512), (1024, 1024, 576), (640, 1408, 1088),
          (128, 128, 512), (256, 384, 576), (512, 1024, 640), (128, 256, 704)]      # a small C


@pytest.mark.parametrize("m,n,k", SHAPES)
def test_gemm_against_float64(m, n, k):
    print(f"gemm {m}x{n}x{k}", flush=True)
    rng = np.random.default_rng(m + 3 * n + 7 * k)
    a = po.bf16_bits(rng.standard_normal((m, k)).astype(np.float32))
    b = po.bf16_bits(rng.standard_normal((n, k)).astype(np.float32))
    da, db, dc = harness.DevBuf(2 * m * k), harness.DevBuf(2 * n * k), harness.DevBuf(2 * m * n + 4096)
    da.upload(a)
    db.upload(b)
    ref, ref_abs = po.gemm_bf16(a, b)
    # f32 sums of K products in any order: K 2^-23 sum |a||b|; one rounding to bf16: 2^-8 |c|
    bound = k * 2.0 ** -23 * ref_abs + 2.0 ** -8 * np.abs(ref) + 1e-30
    first = None
    for _ in range(3):       # the same bits each time: nothing depends on the order in which waves arrive
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


def test_gemm_with_rows_beyond_32_bit_offsets():
    """K past 2^22: rows of A and B are zero but for columns at the beginning, in the middle and at the end."""
    m = n = 128
    k = (1 << 22) + 64
    print(f"gemm {m}x{n}x{k}", flush=True)
    rng = np.random.default_rng(5)
    at = [0, 63, 64, 1 << 21, (1 << 22) - 1, 1 << 22, k - 1]
    cols_a = po.bf16_bits(rng.standard_normal((m, len(at))).astype(np.float32))
    cols_b = po.bf16_bits(rng.standard_normal((n, len(at))).astype(np.float32))
    bufs = []
    for cols in (cols_a, cols_b):
        full = np.zeros((128, k), dtype=np.uint16)
        full[:, at] = cols
        d = harness.DevBuf(2 * 128 * k)
        d.upload(full)
        bufs.append(d)
        del full
    dc = harness.DevBuf(2 * m * n)
    B.proxy_gemm_bf16(bufs[0].ptr, bufs[1].ptr, dc.ptr, m, n, k, 0)
    harness.synchronize()
    got = po.bf16_to_f64(gu.download(dc).view(np.uint16).reshape(m, n))
    ref, ref_abs = po.gemm_bf16(cols_a, cols_b)
    assert np.all(np.abs(got - ref) <= len(at) * 2.0 ** -23 * ref_abs + 2.0 ** -8 * np.abs(ref) + 1e-30)
    for x in bufs + [dc]:
        x.free()


# with 64-bit addresses, by the form that they take (tests/test_host_gemm_forms.py asks the choice itself)
WIDE_K = (1 << 22) + 64
WIDE_FORMS = {
    "256x256": [(3840, 3712)],
    "224x256": [(3072, 4096)],
    "256x192": [(3072, 3200)],
    "160x256": [(2432, 2560)],
    "192x128 by 2": [(1792, 2816)],
    "160x128": [(2176, 2048)],
    "128x128": [(1536, 2048)],
    "128x96": [(1280, 1664)],
    "64x128 by 2": [(896, 1664)],
    "96x64 by 2": [(1152, 1024)],
    "64x64 by 2": [(640, 1280)],
    "32x64 K/4": [(384, 768)],
    "32x32 K/4": [(256, 384)],
}


@pytest.mark.parametrize("m,n", [shape for shapes in WIDE_FORMS.values() for shape in shapes])
def test_gemm_tiles_with_rows_beyond_32_bit_offsets(m, n):
    """K past 2^22: rows of A and B are zero but for eight columns in each of a few places, that of the first, of the last
    and of an odd step of K among them."""
    k = WIDE_K
    print(f"gemm {m}x{n}x{k}", flush=True)
    rng = np.random.default_rng(m + n)
    at = [0, 5 * 64 + 24, (1 << 21) + 8, (1 << 22) - 8, (1 << 22) + 56]
    cols, bufs = [], []
    for rows in (m, n):
        c = po.bf16_bits(rng.standard_normal((rows, 8 * len(at))).astype(np.float32))
        d = harness.DevBuf(2 * rows * k)
        B.proxy_device_fill_async(d.ptr, 0, d.nbytes, 0)
        harness.synchronize()
        for r in range(rows):
            for i, col in enumerate(at):
                B.proxy_copy_h2d(d.ptr + 2 * (r * k + col), c[r, 8 * i:].ctypes.data, 16)
        cols.append(c)
        bufs.append(d)
    dc = harness.DevBuf(2 * m * n + 4096)
    B.proxy_device_fill_async(dc.ptr, 0xEE, dc.nbytes, 0)
    B.proxy_gemm_bf16(bufs[0].ptr, bufs[1].ptr, dc.ptr, m, n, k, 0)
    harness.synchronize()
    out = gu.download(dc)
    assert np.all(out[2 * m * n:] == 0xEE)
    got = po.bf16_to_f64(out[:2 * m * n].view(np.uint16).reshape(m, n))
    ref, ref_abs = po.gemm_bf16(*cols)
    # f32 sums of 40 products that are not zero; one rounding to bf16
    assert np.all(np.abs(got - ref) <= 40 * 2.0 ** -23 * ref_abs + 2.0 ** -8 * np.abs(ref) + 1e-30)
    for x in bufs + [dc]:
        x.free()
