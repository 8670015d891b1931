"""Lists around the number of tensors that a launch of a long list takes (1280), the last launch with arguments of each size, against the
oracle's data region."""
import numpy as np
import pytest

from paper_2406_10707_amd import binding as B
from paper_2406_10707_amd import harness
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
