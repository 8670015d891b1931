"""Restores into tensors of sizes around the scatter kernel's words, groups and tiles, at every misalignment: the tensors' bytes come
back and the bytes between them stay as they are."""
import numpy as np
import pytest

from oracle import readback as rb
from paper_2406_10707_amd import binding as B
from paper_2406_10707_amd import harness, shards
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu
MIB = 1 << 20
SIZES = [1, 15, 16, 17, 1023, 1024, 1025, 2047, 2048, 2049, 4095, 4097, 8191, 8192, 8193, 15361, 16385, 32767, 32768, 32769, 65536 + 1025]


@pytest.mark.parametrize("gap", [1, 3])
@pytest.mark.parametrize("large", [0, 5 * MIB + 3])        # small regions alone, and behind a large tensor
def test_restored_bytes_and_the_bytes_between(tmp_path, gap, large):
    print(f"scatter edges, gap {gap}, large {large}", flush=True)
    tensors, off = [], 0
    for k, n in enumerate(([large] if large else []) + SIZES * 3):
        tensors.append(shards.TensorSpec(f"t{k}", shards.U8, (n,), buffer=0, offset=off, role="raw"))
        off += n + gap + k % 5
    shard, stream = harness.DeviceShard(shards.ShardSpec("edges", 7, tensors, flat_buffers=[(off + 255) // 256 * 256])), harness.Stream()
    shard.fill_device(stream)
    stream.synchronize()
    want = gu.readback_all(shard)
    ck = B.Checkpointer(B.make_config(out_dir=str(tmp_path), dma_chunk_bytes=16 * MIB, pack_superchunk_bytes=16 * MIB, host_ring_bytes=32 * MIB))
    ck.register_tensors(shard.descs())
    ck.snapshot_async(1, stream.cuda_stream)
    ck.wait_immutable_window_end(stream.cuda_stream)
    ck.flush()
    lo, hi = min(shard.ptrs), max(p + t.nbytes for p, t in zip(shard.ptrs, tensors))
    for _ in range(3):
        B.proxy_device_fill_async(lo, 0xEE, hi - lo, stream.handle)
        assert ck.restore(ck.file_name(1), stream.cuda_stream) == 1
        stream.synchronize()
        expect = np.full(hi - lo, 0xEE, dtype=np.uint8)
        for p, w in zip(shard.ptrs, want):
            expect[p - lo:p - lo + w.nbytes] = w
        assert np.array_equal(rb.d2h(lo, hi - lo), expect)
    ck.destroy()
    shard.free()
