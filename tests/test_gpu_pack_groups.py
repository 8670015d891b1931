"""Lists around the sizes of the pack kernel's arguments (32, 128 and 320 tensors), with few and with enough pages for the
look-up by groups (1024), with too many of them in one tensor (off the lines more than 2048, on them more than 16384), one tensor much larger than the
others and not, against the oracle's data region."""
import numpy as np
import pytest

from oracle import oracle
from paper_2406_10707_amd import binding as B
from paper_2406_10707_amd import harness, shards
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 32, 33, 128, 129, 320])
@pytest.mark.parametrize("pages", [1023, 1024, 1025, 2500, 17500])
def test_image_around_the_sizes(n, pages):
    print(f"pack groups, {n} tensors, {pages} pages", flush=True)
    for first in (True, False):          # the large tensor at either end of the list
        sizes = [4096 * (k % 3) + 1 + 977 * k % 4096 for k in range(n - 1)]
        sizes.insert(0 if first else n - 1, 4096 * (pages - sum(-(-s // 4096) for s in sizes)) - 7)
        tensors, off = [], 0
        for k, s in enumerate(sizes):
            off = (off + 15) // 16 * 16 + (k % 16 if pages == 2500 else 0)
            tensors.append(shards.TensorSpec(f"t{k}", shards.U8, (s,), buffer=0, offset=off, role="raw"))
            off += s
        shard, stream = harness.DeviceShard(shards.ShardSpec("groups", n, tensors, flat_buffers=[(off + 255) // 256 * 256])), harness.Stream()
        shard.fill_device(stream)
        stream.synchronize()
        ots = shard.oracle_tensors(gu.readback_all(shard))
        want = np.frombuffer(oracle.serialize_bytes(ots, 0), dtype=np.uint8)[oracle.header_bytes(ots):]
        assert want.nbytes == 4096 * pages
        dst = harness.DevBuf(want.nbytes + 32)
        B.proxy_device_fill_async(dst.ptr, 0xEE, dst.nbytes, stream.handle)
        B.pack_image_noalloc(shard.descs(), dst.ptr + 16, want.nbytes, stream.cuda_stream)
        stream.synchronize()
        got = gu.download(dst)
        assert np.array_equal(got[16:-16], want) and np.all(got[:16] == 0xEE) and np.all(got[-16:] == 0xEE)
        dst.free()
        shard.free()
