"""The Adam step where its blocks are more than the chip has room for at once (2^21 elements) and where they are an eighth more (from there
on they are launched with shared memory that limits how many run beside each other), and its rounding to bf16 in whole quads and in the tail."""
import numpy as np
import pytest

from oracle import proxy_oracle as po
from paper_2406_10707_amd import binding as B
from paper_2406_10707_amd import harness
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


def _bufs(n):
    return [harness.DevBuf(es * n) for es in (2, 4, 4, 4)]


def _read(bufs):
    harness.synchronize()
    return [gu.download(b).view(dt) for b, dt in zip(bufs, (np.uint16, np.float32, np.float32, np.float32))]


@pytest.mark.parametrize("numel", [4 * 64 * 8192, 4 * 64 * 8192 + 1, 4 * 64 * 8192 + 7, 4 * 64 * 9216, 4 * 64 * 9216 + 1, 4 * 64 * 9216 + 7])
def test_adam_around_a_full_chip(numel):
    print(f"adam numel {numel}", flush=True)
    bufs = _bufs(numel)
    B.proxy_fill_state(*[b.ptr for b in bufs], numel, 11, 2, 0)
    _, w0, m0, v0 = _read(bufs)
    B.proxy_adam_step(*[b.ptr for b in bufs], numel, 11, 2, 3, 0)
    gp, gw, gm, gv = _read(bufs)
    ow, om, ov, _ = po.adam_step(w0.astype(np.float64), m0.astype(np.float64), v0.astype(np.float64), 11, 2, 3)
    # about ten float32 operations per element, as in the test of the update's arithmetic
    assert np.max(np.abs(gm - om)) <= 1e-5 * np.max(np.abs(om)) + 1e-12
    assert np.max(np.abs(gv - ov)) <= 1e-5 * np.max(np.abs(ov)) + 1e-18
    assert np.all(np.abs(gw - ow) <= 1e-5 * (np.abs(w0) + np.abs(ow - w0)) + 1e-12)
    assert np.array_equal(gp, po.bf16_bits(gw))


def test_bf16_of_every_kind_of_value():
    """Every upper half of an f32 with lower halves at and around the tie: NaN payloads, infinities, denormals, carries into
    the exponent. With lr = 0 the update leaves the weights as they are (a NaN becomes a quiet one, and
    -0 - 0 m is +0 for negative m)."""
    hi = np.arange(65536, dtype=np.uint32) << 16
    words = (hi[:, None] | np.array([0, 1, 0x7FFF, 0x8000, 0x8001, 0xFFFF], dtype=np.uint32)).reshape(-1)
    words = np.concatenate([words, words[-2:], words[6 * 0x7FC0:6 * 0x7FC0 + 1]])       # a tail of three: negative NaNs, a NaN
    n = words.size
    assert n % 4 == 3
    bufs = _bufs(n)
    zeros = np.zeros(n, dtype=np.float32)
    for b, x in zip(bufs[1:], (words, zeros, zeros)):
        b.upload(x)
    B.proxy_adam_step(*[b.ptr for b in bufs], n, 11, 2, 1, 0, lr=0.0)
    gp, gw, _, _ = _read(bufs)
    nan = (words & 0x7FFFFFFF) > 0x7F800000
    assert np.array_equal(gw[~nan], words.view(np.float32)[~nan]) and np.all(np.isnan(gw[nan]))
    assert np.array_equal(gp, po.bf16_bits(gw))
