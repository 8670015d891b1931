"""Snapshots of a shard that is written straight into its ring slot while its pair holds (3.4 MiB) and through staging when it does not
(5.1 MiB), in turn and with only stream order between them, against the oracle."""
import numpy as np
import pytest

from oracle import oracle
from paper_2406_10707_amd import binding as B
from paper_2406_10707_amd import harness, shards
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu
MIB = 1 << 20


@pytest.mark.parametrize("turns", [[0, 1, 0, 1, 0, 1], [1, 1, 0, 0, 1, 0]])
def test_straight_and_staged_in_turn(tmp_path, turns):
    print(f"straight and staged in turn {turns}", flush=True)
    n = 890_001
    spec = shards.ShardSpec("turns", 1, [shards.TensorSpec("p", shards.BF16, (n,), buffer=0, offset=0, role="p_bf16"),
                                         shards.TensorSpec("w", shards.F32, (n,), buffer=1, offset=0, role="master")],
                            flat_buffers=[2 * MIB, 4 * MIB])
    shard, stream = harness.DeviceShard(spec), harness.Stream()
    w = np.random.default_rng(1).integers(0, 1 << 16, n).astype(np.uint32) << 16       # f32 values that bf16 holds
    w[(w & 0x7F800000) == 0x7F800000] = 0x3F800000
    p = (w >> 16).astype(np.uint16)
    good = harness.DevBuf(p.nbytes)
    for dst, src in ((shard.ptrs[0], p), (good.ptr, p), (shard.ptrs[1], w)):
        B.proxy_copy_h2d(dst, src.ctypes.data, src.nbytes)
    ck = B.Checkpointer(B.make_config(out_dir=str(tmp_path), dma_chunk_bytes=16 * MIB, pack_superchunk_bytes=16 * MIB, host_ring_bytes=32 * MIB))
    ck.declare_derived([(0, 1)])
    ck.register_tensors(shard.descs())
    for it, broken in enumerate(turns, 1):
        ck.wait_immutable_window_end(stream.cuda_stream)
        B.proxy_copy_d2d_async(shard.ptrs[0], good.ptr, p.nbytes, stream.handle)
        if broken:
            B.proxy_device_fill_async(shard.ptrs[0] + 2 * (n - 1 - it), 0x5A, 2, stream.handle)
        ck.snapshot_async(it, stream.cuda_stream)
    ck.wait_immutable_window_end(stream.cuda_stream)
    ck.flush()
    for it, broken in enumerate(turns, 1):
        q = p.copy()
        if broken:
            q[n - 1 - it] = 0x5A5A
        want, version = oracle.serialize_bytes_v2(shard.oracle_tensors([q.view(np.uint8), w.view(np.uint8)]), it, [(0, 1)])
        assert version == 2 - broken and open(ck.file_name(it), "rb").read() == want
        st = ck.stats(it)
        assert st["d2h_done"] == 1 and st["committed"] == 1 and 0 < st["d2h_span_ms"] <= st["request_to_d2h_end_ms"]
    for it in (len(turns), turns.index(1) + 1, turns.index(0) + 1):
        shard.poison()
        assert ck.restore(ck.file_name(it), stream.cuda_stream) == it
        stream.synchronize()
        q = p.copy()
        if turns[it - 1]:
            q[n - 1 - it] = 0x5A5A
        got = gu.readback_all(shard)
        assert np.array_equal(got[0], q.view(np.uint8)) and np.array_equal(got[1], w.view(np.uint8))
    ck.destroy()
    good.free()
    shard.free()
