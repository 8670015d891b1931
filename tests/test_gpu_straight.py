"""Data regions around the size up to which the pack kernel writes the ring slot itself (4 MiB), update and snapshot in every
iteration with only stream order between them, against the oracle."""
import numpy as np
import pytest

from oracle import oracle
from paper_2406_10707_amd import binding as B
from paper_2406_10707_amd import harness, shards
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu
MIB = 1 << 20


@pytest.mark.parametrize("sizes", [[1], [4096], [4 * MIB - 4096, 4096], [4 * MIB], [4 * MIB - 4096, 4097], [4 * MIB + 1], [100003, 7, 2 * MIB + 5]])
@pytest.mark.parametrize("policy", [B.CKPT_WINDOW_D2H, B.CKPT_WINDOW_PACK])
def test_snapshots_every_iteration(tmp_path, sizes, policy):
    print(f"straight {sizes} policy {policy}", flush=True)
    tensors, off = [], 0
    for k, n in enumerate(sizes):
        tensors.append(shards.TensorSpec(f"t{k}", shards.U8, (n,), buffer=0, offset=off, role="raw"))
        off += n + k + 1
    shard = harness.DeviceShard(shards.ShardSpec("straight", 3, tensors, flat_buffers=[(off + 255) // 256 * 256]))
    stream = harness.Stream()
    ck = B.Checkpointer(B.make_config(out_dir=str(tmp_path), dma_chunk_bytes=16 * MIB, pack_superchunk_bytes=16 * MIB, host_ring_bytes=32 * MIB,
                                      window_policy=policy))
    ck.register_tensors(shard.descs())
    shard.fill_device(stream)
    clones = {}
    for it in range(1, 7):
        ck.wait_immutable_window_end(stream.cuda_stream)
        shard.update(it, stream)
        clones[it] = shard.clone_all(stream)
        ck.snapshot_async(it, stream.cuda_stream)
    ck.flush()
    stream.synchronize()
    for it, bufs in clones.items():
        want = [gu.download(b) for b in bufs]
        assert oracle.compare_file(shard.oracle_tensors(want), it, ck.file_name(it)) is None
        st = ck.stats(it)
        assert st["d2h_done"] == 1 and st["committed"] == 1 and st["pack_launches"] == 1 and st["request_to_d2h_end_ms"] >= 0
    shard.poison()
    assert ck.restore(ck.file_name(6), stream.cuda_stream) == 6
    stream.synchronize()
    assert all(np.array_equal(a, b) for a, b in zip(want, gu.readback_all(shard)))
    ck.destroy()
    shard.free()
