"""Chunks that go between ring slot and file in several pieces (4 MiB each): sizes around the pieces' and the chunks' ends, a
ring smaller than the shard, the sinks, tensors copied directly (their segments are cut by the pieces on restore)."""
import numpy as np
import pytest

from oracle import oracle
from paper_2406_10707_amd import binding as B
from paper_2406_10707_amd import harness, shards
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu
MIB = 1 << 20


@pytest.mark.parametrize("sizes,chunk,options", [
    ([4 * MIB], 16 * MIB, {}),
    ([4 * MIB + 1], 16 * MIB, {}),
    ([16 * MIB - 4096, 5], 16 * MIB, {}),
    ([3, 16 * MIB, 20 * MIB + 7, 11, 33 * MIB], 16 * MIB, {}),
    ([3, 16 * MIB, 20 * MIB + 7, 11, 33 * MIB], 16 * MIB, {"io_mode": B.CKPT_IO_PWRITE}),
    ([3, 16 * MIB, 20 * MIB + 7, 11, 33 * MIB], 16 * MIB, {"keep_last": 1, "prealloc_files": 2, "n_io_threads": 1}),
    ([3, 16 * MIB, 20 * MIB + 7, 11, 33 * MIB], 16 * MIB, {"direct_min_bytes": 4 * MIB}),
    ([70 * MIB + 13, 1], 64 * MIB, {"n_io_threads": 7}),
    ([3, 16 * MIB, 20 * MIB + 7, 11, 33 * MIB], 16 * MIB, {"pack_superchunk_bytes": 64 * MIB}),       # the first chunk packed apart
])
def test_snapshot_and_restore(tmp_path, sizes, chunk, options):
    print(f"pieces {sizes} chunk {chunk} {options}", flush=True)
    tensors, off = [], 0
    for k, n in enumerate(sizes):
        tensors.append(shards.TensorSpec(f"t{k}", shards.U8, (n,), buffer=0, offset=off, role="raw"))
        off += n + 2 * k + 1
    shard = harness.DeviceShard(shards.ShardSpec("pieces", 3, tensors, flat_buffers=[(off + 255) // 256 * 256]))
    stream = harness.Stream()
    ck = B.Checkpointer(B.make_config(**{"out_dir": str(tmp_path), "dma_chunk_bytes": chunk, "pack_superchunk_bytes": 2 * chunk, "host_ring_bytes": 2 * chunk, **options}))
    ck.register_tensors(shard.descs())
    shard.fill_device(stream)
    for it in (1, 2, 3):
        shard.update(it, stream)
        ck.snapshot_async(it, stream.cuda_stream)
        ck.wait_immutable_window_end(stream.cuda_stream)
        ck.flush(it)
        want = gu.readback_all(shard)
        assert oracle.compare_file(shard.oracle_tensors(want), it, ck.file_name(it)) is None
    for _ in range(2):
        shard.poison()
        assert ck.restore(ck.file_name(3), stream.cuda_stream) == 3
        stream.synchronize()
        got = gu.readback_all(shard)
        assert all(np.array_equal(a, b) for a, b in zip(want, got))
    ck.destroy()
    shard.free()
