"""The Adam step where its grid ends: one lane, the last lane of a block, one beyond it, a tail behind whole quads; nothing
outside the tensors is touched. Against the float64 oracle."""
import zlib

import numpy as np
import pytest

from oracle import proxy_oracle as po
from paper_2406_10707_amd import binding as B
from paper_2406_10707_amd import harness
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("numel", [1, 3, 4, 5, 255, 256, 257, 259, 1023, 65536 + 2])
def test_adam_at_the_edges_of_its_grid(numel):
    print(f"adam numel {numel}", flush=True)
    guard = 64
    bufs = [harness.DevBuf(es * numel + 2 * guard) for es in (2, 4, 4, 4)]
    for b in bufs:
        B.proxy_device_fill_async(b.ptr, 0xEE, b.nbytes, 0)
    ptrs = [b.ptr + guard for b in bufs]
    B.proxy_fill_state(*ptrs, numel, 11, 2, 0)
    harness.synchronize()

    def read():
        out = []
        for b, es, dt in zip(bufs, (2, 4, 4, 4), (np.uint16, np.float32, np.float32, np.float32)):
            raw = gu.download(b)
            assert np.all(raw[:guard] == 0xEE) and np.all(raw[guard + es * numel:] == 0xEE)
            out.append(raw[guard:guard + es * numel].copy().view(dt))
        return out

    _, w0, m0, v0 = read()
    B.proxy_adam_step(*ptrs, numel, 11, 2, 3, 0)
    harness.synchronize()
    gp, gw, gm, gv = read()
    ow, om, ov, _ = po.adam_step(w0.astype(np.float64), m0.astype(np.float64), v0.astype(np.float64), 11, 2, 3)
    # about ten float32 operations per element, as in the test of the update's arithmetic
    assert np.max(np.abs(gm - om)) <= 1e-5 * np.max(np.abs(om)) + 1e-12
    assert np.max(np.abs(gv - ov)) <= 1e-5 * np.max(np.abs(ov)) + 1e-18
    assert np.all(np.abs(gw - ow) <= 1e-5 * (np.abs(w0) + np.abs(ow - w0)) + 1e-12)
    assert np.array_equal(gp, po.bf16_bits(gw))


def _after_three_steps(n):
    """Outputs of three steps from states whose elements depend on their index alone."""
    u = ((np.arange(3 * 65538, dtype=np.uint64) * np.uint64(2654435761)) & np.uint64(0xFFFFFFFF)).astype(np.uint32).reshape(3, -1)[:, :n] >> 8
    state = [u[k].astype(np.float32) * np.float32(s) for k, s in enumerate((2.0 ** -29, -2.0 ** -31, 2.0 ** -44))]
    bufs = [harness.DevBuf(es * n) for es in (2, 4, 4, 4)]
    for b, x in zip(bufs[1:], state):
        b.upload(x)
    harness.synchronize()
    for step in (1, 2, 3):
        B.proxy_adam_step(*[b.ptr for b in bufs], n, 11, 2, step, 0)
    harness.synchronize()
    return [gu.download(b) for b in bufs]


@pytest.mark.parametrize("numel,sums", [
    (65538, [0x62b7252e, 0x2ce87695, 0x81f84e75, 0x81b6bda4]),
    (5001, [0xfafc16ef, 0xd7d5fcdb, 0x7349a75f, 0x42fb9f57]),
    (1027, [0x5b6aaddb, 0x6408be73, 0x5d371b2d, 0x7467786d]),
    (3, [0x1cb869ba, 0x199d9b8f, 0xd913ff1c, 0x0ac74c9a]),
])
def test_adam_bits(numel, sums):
    """The bits that the grid-stride form of this kernel gave, in whole quads and in the tail (checksums taken from it)."""
    print(f"adam bits {numel}", flush=True)
    assert [zlib.crc32(x.tobytes()) for x in _after_three_steps(numel)] == sums
