"""A snapshot's last chunks, which are shared among the copy streams in parts of 16 MiB: one to five chunks, the last one a page,
part of a part, whole parts; one, two and three streams; tensors copied directly and host-resident objects among the parts; a second
snapshot while the first one may still be on its way to the file. The same files restored, over the streams in turn."""
import numpy as np
import pytest

from oracle import oracle
from paper_2406_10707_amd import binding as B
from paper_2406_10707_amd import harness, shards
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu
MIB = 1 << 20


@pytest.mark.parametrize("sizes,chunk,options", [
    ([32 * MIB], 32 * MIB, {}),
    ([32 * MIB, 1], 32 * MIB, {}),
    ([5, 48 * MIB - 4096], 32 * MIB, {"keep_last": 1, "prealloc_files": 2}),
    ([64 * MIB + 17, 3], 32 * MIB, {"n_dma_streams": 3}),
    ([20 * MIB + 7] * 4, 32 * MIB, {"n_dma_streams": 1}),
    ([30 * MIB + 1, 7, 90 * MIB, 9], 32 * MIB, {}),
    ([30 * MIB + 1, 7, 90 * MIB, 9], 32 * MIB, {"direct_min_bytes": 4 * MIB}),
    ([30 * MIB + 1, 7, 90 * MIB, 9], 32 * MIB, {"io_mode": B.CKPT_IO_PWRITE, "n_io_threads": 2}),
    ([30 * MIB + 1, 7, 90 * MIB, 9], 20 * MIB, {"pack_superchunk_bytes": 160 * MIB}),       # the first chunk packed apart
    ([30 * MIB + 1, 7, 20 * MIB], 20 * MIB, {"pack_superchunk_bytes": 160 * MIB}),          # the same, and among the last
    ([30 * MIB + 1, 7, 90 * MIB, 9], 64 * MIB, {"window_policy": B.CKPT_WINDOW_PACK, "dev_staging_bytes": 256 * MIB}),
])
def test_snapshots_and_restore(tmp_path, sizes, chunk, options):
    print(f"parts {sizes} chunk {chunk} {options}", flush=True)
    tensors, off = [], 0
    for k, n in enumerate(sizes):
        tensors.append(shards.TensorSpec(f"t{k}", shards.U8, (n,), buffer=0, offset=off, role="raw"))
        off += n + 2 * k + 1
    shard = harness.DeviceShard(shards.ShardSpec("parts", 4, tensors, flat_buffers=[(off + 255) // 256 * 256]))
    stream = harness.Stream()
    ck = B.Checkpointer(B.make_config(**{"out_dir": str(tmp_path), "dma_chunk_bytes": chunk, "pack_superchunk_bytes": 2 * chunk, "host_ring_bytes": 2 * chunk, **options}))
    ck.register_tensors(shard.descs())
    shard.fill_device(stream)
    for it in (1, 3, 5):
        wants = {}
        for i in (it, it + 1):      # the second one is requested as soon as the first one's window has closed
            shard.update(i, stream)
            ck.snapshot_async(i, stream.cuda_stream)
            ck.wait_immutable_window_end(stream.cuda_stream)
            stream.synchronize()
            wants[i] = gu.readback_all(shard)
        for i, want in wants.items():
            ck.flush(i)
            if i == it and options.get("keep_last"):
                continue        # this file has been overwritten by the next one
            assert oracle.compare_file(shard.oracle_tensors(want), i, ck.file_name(i)) is None
    for _ in range(2):
        shard.poison()
        assert ck.restore(ck.file_name(6), stream.cuda_stream) == 6
        stream.synchronize()
        assert all(np.array_equal(a, b) for a, b in zip(wants[6], gu.readback_all(shard)))
    ck.destroy()
    shard.free()


def test_many_chunks_of_more_than_64_mib(tmp_path):
    """Eight chunks of 72 MiB: the last ones are not shared, and a restore sends those in between as a whole while the link is busy."""
    print("eight chunks of 72 MiB", flush=True)
    sizes = [200 * MIB + 5, 3, 150 * MIB, 180 * MIB + 4097]
    tensors, off = [], 0
    for k, n in enumerate(sizes):
        tensors.append(shards.TensorSpec(f"t{k}", shards.U8, (n,), buffer=0, offset=off, role="raw"))
        off += n + 2 * k + 1
    shard = harness.DeviceShard(shards.ShardSpec("parts", 4, tensors, flat_buffers=[(off + 255) // 256 * 256]))
    stream = harness.Stream()
    ck = B.Checkpointer(B.make_config(out_dir=str(tmp_path), dma_chunk_bytes=72 * MIB, pack_superchunk_bytes=144 * MIB, host_ring_bytes=288 * MIB))
    ck.register_tensors(shard.descs())
    shard.fill_device(stream)
    ck.snapshot_async(1, stream.cuda_stream)
    ck.wait_immutable_window_end(stream.cuda_stream)
    stream.synchronize()
    want = gu.readback_all(shard)
    ck.flush(1)
    assert oracle.compare_file(shard.oracle_tensors(want), 1, ck.file_name(1)) is None
    for _ in range(2):
        shard.poison()
        assert ck.restore(ck.file_name(1), stream.cuda_stream) == 1
        stream.synchronize()
        assert all(np.array_equal(a, b) for a, b in zip(want, gu.readback_all(shard)))
    ck.destroy()
    shard.free()
