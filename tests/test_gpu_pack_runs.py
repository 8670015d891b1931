"""Lists large enough for the pack kernel's other block order, off the 128-byte lines and, for more or less than half of
their pages, on them, against the oracle's data region; the last block of 64 is whole, nearly empty, or one short."""
import numpy as np
import pytest

from oracle import oracle
from paper_2406_10707_amd import binding as B
from paper_2406_10707_amd import harness, shards
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes,leads", [
    ([2048 * 4096], [2]), ([2049 * 4096 - 5], [6]), ([2047 * 4096], [2]), ([(2048 + 15) * 4096 + 1], [14]),
    ([3000001, 6000002, 4000003, 5000004], [126, 0, 64, 4]), ([9000001, 3000002], [0, 2]), ([1 << 20] * 9 + [12345] * 9, [2, 0, 130] * 6)])
def test_image_of_a_large_list(sizes, leads):
    print(f"pack runs, {len(sizes)} tensors", flush=True)
    tensors, off = [], 0
    for k, (n, lead) in enumerate(zip(sizes, leads)):
        off = (off + 255) // 256 * 256 + lead
        tensors.append(shards.TensorSpec(f"t{k}", shards.U8, (n,), buffer=0, offset=off, role="raw"))
        off += n
    shard, stream = harness.DeviceShard(shards.ShardSpec("runs", 5, tensors, flat_buffers=[(off + 255) // 256 * 256])), harness.Stream()
    shard.fill_device(stream)
    stream.synchronize()
    ots = shard.oracle_tensors(gu.readback_all(shard))
    want = np.frombuffer(oracle.serialize_bytes(ots, 0), dtype=np.uint8)[oracle.header_bytes(ots):]
    dst = harness.DevBuf(want.nbytes + 32)
    for call in (B.pack_image, B.pack_image_noalloc):
        B.proxy_device_fill_async(dst.ptr, 0xEE, dst.nbytes, stream.handle)
        call(shard.descs(), dst.ptr + 16, want.nbytes, stream.cuda_stream)
        stream.synchronize()
        got = gu.download(dst)
        assert np.array_equal(got[16:-16], want) and np.all(got[:16] == 0xEE) and np.all(got[-16:] == 0xEE)
    dst.free()
    shard.free()
