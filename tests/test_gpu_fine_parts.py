"""Snapshots of one chunk, whose copies go in up to twelve parts, the first one half as long: around the smallest size that is copied at
all (4 MiB and a page), where the parts begin to grow with the chunk, and where they reach 16 MiB; and small ones, which the pack kernel stores over the link and
several I/O threads write. Files against the oracle; a snapshot requested while the one before is still being written takes the other way."""
import numpy as np
import pytest

from oracle import oracle
from paper_2406_10707_amd import binding as B
from paper_2406_10707_amd import harness, shards
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu
MIB = 1 << 20


@pytest.mark.parametrize("sizes,chunk,options", [
    ([2 * MIB], 64 * MIB, {}),                                   # straight: one piece more than a quarter each
    ([2 * MIB + 1, 5], 8 * MIB, {"n_io_threads": 2}),
    ([4 * MIB + 1], 64 * MIB, {}),                               # the smallest copied one
    ([5 * MIB + 4095, 3], 8 * MIB, {"keep_last": 1, "prealloc_files": 2}),
    ([22 * MIB - 4096], 64 * MIB, {}),                           # eleven times 2 MiB: the last with parts of 2 MiB
    ([22 * MIB], 64 * MIB, {"n_dma_streams": 3}),
    ([22 * MIB + 4096, 7], 64 * MIB, {"n_dma_streams": 1}),      # one stream: a single copy
    ([9 * MIB + 1, 7, 31 * MIB + 5], 64 * MIB, {"direct_min_bytes": 4 * MIB}),
    ([9 * MIB + 1, 7, 31 * MIB + 5], 64 * MIB, {"window_policy": B.CKPT_WINDOW_PACK, "io_mode": B.CKPT_IO_PWRITE}),
    ([165 * MIB - 8192], 192 * MIB, {}),                         # eleven times 15 MiB
    ([165 * MIB], 192 * MIB, {}),                                # parts of 16 MiB, all alike
])
def test_snapshots_of_one_chunk(tmp_path, sizes, chunk, options):
    print(f"fine parts {sizes} chunk {chunk} {options}", flush=True)
    tensors, off = [], 0
    for k, n in enumerate(sizes):
        tensors.append(shards.TensorSpec(f"t{k}", shards.U8, (n,), buffer=0, offset=off, role="raw"))
        off += n + 2 * k + 1
    shard = harness.DeviceShard(shards.ShardSpec("fine", 4, tensors, flat_buffers=[(off + 255) // 256 * 256]))
    stream = harness.Stream()
    ck = B.Checkpointer(B.make_config(**{"out_dir": str(tmp_path), "dma_chunk_bytes": chunk, "pack_superchunk_bytes": chunk, "host_ring_bytes": 2 * chunk, **options}))
    ck.register_tensors(shard.descs())
    assert ck.layout()["n_chunks"] == 1
    shard.fill_device(stream)
    wants = {}
    for it in (1, 2):           # the second one is requested as soon as the first one's window has closed
        shard.update(it, stream)
        ck.snapshot_async(it, stream.cuda_stream)
        ck.wait_immutable_window_end(stream.cuda_stream)
        stream.synchronize()
        wants[it] = gu.readback_all(shard)
    for it in (1, 2):
        ck.flush(it)
        if it == 2 or not options.get("keep_last"):
            assert oracle.compare_file(shard.oracle_tensors(wants[it]), it, ck.file_name(it)) is None
    shard.poison()
    assert ck.restore(ck.file_name(2), stream.cuda_stream) == 2
    stream.synchronize()
    assert all(np.array_equal(a, b) for a, b in zip(wants[2], gu.readback_all(shard)))
    ck.destroy()
    shard.free()
