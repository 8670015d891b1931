"""Snapshots of one chunk: small ones, which the pack kernel stores over the link; from the smallest size that is copied at all (4 MiB and a
page) up to 64 MiB in one copy; larger ones in a copy for every 64 MiB begun. Pieces that the I/O threads share evenly, one thread and more. Files
against the oracle; the second snapshot is requested with only stream order between it and the first, whose file may still be on its way (copies are
then not shared out)."""
import numpy as np
import pytest

from oracle import oracle
from paper_2406_10707_amd import binding as B
from paper_2406_10707_amd import harness, shards
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu
MIB = 1 << 20


@pytest.mark.parametrize("sizes,chunk,options", [
    ([2 * MIB], 64 * MIB, {}),                                   # straight: four pieces of half a MiB
    ([2 * MIB + 1, 5], 8 * MIB, {"n_io_threads": 2}),
    ([700_001], 8 * MIB, {"n_io_threads": 16}),                  # fewer pieces than threads
    ([4 * MIB + 1], 64 * MIB, {}),                               # the smallest copied one
    ([5 * MIB + 4095, 3], 8 * MIB, {"keep_last": 1, "prealloc_files": 2}),
    ([5 * MIB + 4095, 3], 8 * MIB, {"n_io_threads": 1}),
    ([22 * MIB - 4096], 64 * MIB, {}),
    ([22 * MIB], 64 * MIB, {"n_dma_streams": 3}),
    ([22 * MIB + 4096, 7], 64 * MIB, {"n_dma_streams": 1}),
    ([9 * MIB + 1, 7, 31 * MIB + 5], 64 * MIB, {"direct_min_bytes": 4 * MIB}),
    ([9 * MIB + 1, 7, 31 * MIB + 5], 64 * MIB, {"window_policy": B.CKPT_WINDOW_PACK, "io_mode": B.CKPT_IO_PWRITE}),
    ([64 * MIB], 192 * MIB, {}),                                 # one copy
    ([64 * MIB + 1], 192 * MIB, {}),                             # two
    ([64 * MIB + 1], 192 * MIB, {"n_dma_streams": 1}),           # one stream: a single copy
    ([101 * MIB, 5, 41 * MIB + 77], 192 * MIB, {"direct_min_bytes": 4 * MIB, "n_io_threads": 3}),      # three, cut within both tensors
    ([165 * MIB - 8192], 192 * MIB, {}),
    ([165 * MIB], 192 * MIB, {}),
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
    clones = {}
    for it in (1, 2):
        ck.wait_immutable_window_end(stream.cuda_stream)
        shard.update(it, stream)
        clones[it] = shard.clone_all(stream)
        ck.snapshot_async(it, stream.cuda_stream)
    ck.wait_immutable_window_end(stream.cuda_stream)
    stream.synchronize()
    wants = {it: [gu.download(b) for b in bs] for it, bs in clones.items()}
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
