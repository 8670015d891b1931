"""The Adam step where its grid ends: one lane, the last lane of a block, one beyond it, a tail behind whole quads; nothing
outside the tensors is touched. Against the float64 oracle."""
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
