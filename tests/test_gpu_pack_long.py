"""Lists around the number of tensors that a launch of a long list takes (1280), the last launch with arguments of each size, against the
oracle's data region."""
import numpy as np
import pytest

from paper_2406_10707_amd import binding as B
from paper_2406_10707_amd import harness, shards
from tests import gpu_util as gu
from tests.test_gpu_pack_batch import _shard, _want

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [321, 1279, 1280, 1281, 1313, 1409, 1601, 2561])
def test_image_of_a_long_list(n):
    print(f"pack of a long list, {n} tensors", flush=True)
    shard, stream = _shard(n, n), harness.Stream()
    shard.fill_device(stream)
    stream.synchronize()
    want = _want(shard)
    dst = harness.DevBuf(want.nbytes + 32)
    B.proxy_device_fill_async(dst.ptr, 0xEE, dst.nbytes, stream.handle)
    B.pack_image_noalloc(shard.descs(), dst.ptr + 16, want.nbytes, stream.cuda_stream)
    stream.synchronize()
    got = gu.download(dst)
    assert np.array_equal(got[16:-16], want) and np.all(got[:16] == 0xEE) and np.all(got[-16:] == 0xEE)
    dst.free()
    shard.free()


@pytest.mark.parametrize("nbytes", [2 << 20, (2 << 20) + 1])         # 2 MiB in the mean is the largest that goes in long launches
def test_image_of_a_list_of_large_misaligned_tensors(nbytes):
    print(f"pack of 323 tensors of {nbytes} bytes", flush=True)
    tensors, off = [], 0
    for k in range(323):
        tensors.append(shards.TensorSpec(f"t{k}", shards.U8, (nbytes,), buffer=0, offset=off + 20, role="raw"))
        off += (nbytes + 128 + 127) // 128 * 128
    shard, stream = harness.DeviceShard(shards.ShardSpec("large", 323, tensors, flat_buffers=[off + 256])), harness.Stream()
    shard.fill_device(stream)
    stream.synchronize()
    pages = -(-nbytes // 4096)
    dst = harness.DevBuf(4096 * pages * 323)
    B.proxy_device_fill_async(dst.ptr, 0xEE, dst.nbytes, stream.handle)
    B.pack_image_noalloc(shard.descs(), dst.ptr, dst.nbytes, stream.cuda_stream)
    stream.synchronize()
    got = gu.download(dst).reshape(323, 4096 * pages)
    assert not got[:, nbytes:].any()
    for k in range(323):
        assert np.array_equal(got[k, :nbytes], gu.readback(shard, k)), k
    dst.free()
    shard.free()
