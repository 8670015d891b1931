"""Lists around the number of tensors one launch of the pack kernel takes (320), at every misalignment of the source and
a destination that is 16-byte aligned only, against the oracle's data region; the two entry points overlapping on two
streams, which share nothing."""
import numpy as np
import pytest

from oracle import oracle
from paper_2406_10707_amd import binding as B
from paper_2406_10707_amd import harness, shards
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


def _shard(n, seed):
    sizes = [1, 17, 1023, 1024, 1025, 4095, 4096, 4097, 12345, 32768 + 5]
    tensors, off = [], 0
    for k in range(n):
        off = (off + 15) // 16 * 16 + k % 16
        tensors.append(shards.TensorSpec(f"t{k}", shards.U8, (sizes[k % 10],), buffer=0, offset=off, role="raw"))
        off += sizes[k % 10]
    return harness.DeviceShard(shards.ShardSpec("batch", seed, tensors, flat_buffers=[(off + 255) // 256 * 256]))


def _want(shard):
    ots = shard.oracle_tensors(gu.readback_all(shard))
    return np.frombuffer(oracle.serialize_bytes(ots, 0), dtype=np.uint8)[oracle.header_bytes(ots):]


@pytest.mark.parametrize("n", [1, 319, 320, 321, 641])
def test_image_of_one_and_several_launches(n):
    print(f"pack batch, {n} tensors", flush=True)
    shard, stream = _shard(n, n), harness.Stream()
    shard.fill_device(stream)
    stream.synchronize()
    want = _want(shard)
    dst = harness.DevBuf(want.nbytes + 32)
    for call in (B.pack_image, B.pack_image_noalloc):
        B.proxy_device_fill_async(dst.ptr, 0xEE, dst.nbytes, stream.handle)
        call(shard.descs(), dst.ptr + 16, want.nbytes, stream.cuda_stream)
        stream.synchronize()
        got = gu.download(dst)
        assert np.array_equal(got[16:-16], want) and np.all(got[:16] == 0xEE) and np.all(got[-16:] == 0xEE)
    dst.free()
    shard.free()


def test_overlapping_calls_on_two_streams():
    print("pack batch, two streams", flush=True)
    a, b = _shard(500, 1), _shard(333, 2)
    sa, sb = harness.Stream(), harness.Stream()
    a.fill_device(sa)
    b.fill_device(sb)
    sa.synchronize()
    sb.synchronize()
    wa, wb = _want(a), _want(b)
    da, db = harness.DevBuf(wa.nbytes), harness.DevBuf(wb.nbytes)
    for _ in range(20):
        B.pack_image_noalloc(a.descs(), da.ptr, wa.nbytes, sa.cuda_stream)
        B.pack_image_noalloc(b.descs(), db.ptr, wb.nbytes, sb.cuda_stream)
    sa.synchronize()
    sb.synchronize()
    assert np.array_equal(gu.download(da), wa) and np.array_equal(gu.download(db), wb)
    for x in (a, b, da, db):
        x.free()
