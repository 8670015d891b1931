"""The check and the regeneration of derived tensors on flattened buffers: element counts around a lane's group, a block's
share and a tile, at addresses aligned to the element size only. A single differing element anywhere (first, last, behind the
last whole group, at a block's or a tile's end) must make the snapshot an ordinary version-1 file; without one the file is
version 2 and a restore into overwritten memory brings every bit back, guards between the tensors included."""
import numpy as np
import pytest

from oracle import oracle
from paper_2406_10707_amd import binding as B
from paper_2406_10707_amd import harness, shards
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu
COUNTS = [1, 3, 4, 5, 7, 1023, 1024, 1025, 4095, 4096, 4097, 8191, 8192, 8193, 12289, 20003]
# around a wave's share, small work items in a number that four does not divide
SMALL = [2, 255, 256, 257, 259, 508, 511, 512, 513, 516, 4608, 4609, 8192 + 511]


def _state(shift, counts):
    """Tensors p0, m0, p1, m1, ... in two flat buffers, starts shifted element-wise by up to 15."""
    tensors, off = [], [0, 0]
    for k, n in enumerate(counts):
        for b, (role, code, es) in enumerate((("p_bf16", B.CKPT_BF16, 2), ("master", B.CKPT_F32, 4))):
            off[b] += es * ((k * 5 + shift) % 16)
            tensors.append(shards.TensorSpec(f"t{k}.{role}", code, (n,), buffer=b, offset=off[b], role="raw"))
            off[b] += es * n
    return shards.ShardSpec("pairs", 7, tensors, flat_buffers=[(o + 255) // 256 * 256 + 256 for o in off])


@pytest.mark.parametrize("counts", [COUNTS, SMALL], ids=["counts", "small"])
@pytest.mark.parametrize("shift", [0, 1, 2, 3])
def test_check_and_regeneration(tmp_path, shift, counts):
    print(f"pairs unaligned, shift {shift}", flush=True)
    shard, stream = harness.DeviceShard(_state(shift, counts)), harness.Stream()
    rng = np.random.default_rng(shift)
    for f in shard.flat:
        B.proxy_device_fill_async(f.ptr, 0x5A, f.nbytes, stream.handle)
    stream.synchronize()
    bits = []
    for k, n in enumerate(counts):
        m = (rng.standard_normal(n, dtype=np.float32) * np.float32(0.02))
        special = np.array([0x7FC00001, 0xFFC12345, 0x80000000, 0x00000001, 0x807FFFFF, 0xFFFFFFFF, 0x7F800000, 0x3F808000, 0x3F818000], dtype=np.uint32)
        u = m.view(np.uint32).copy()
        u[rng.integers(0, n, max(1, n // 16))] = special[rng.integers(0, len(special), max(1, n // 16))]
        p = shards.f32_to_bf16_rne(u.view(np.float32))
        bits.append((p, u))
        B.proxy_copy_h2d(shard.ptrs[2 * k], p.ctypes.data, p.nbytes)
        B.proxy_copy_h2d(shard.ptrs[2 * k + 1], u.ctypes.data, u.nbytes)
    ck = B.Checkpointer(B.make_config(out_dir=str(tmp_path), dma_chunk_bytes=64 << 10, pack_superchunk_bytes=256 << 10, host_ring_bytes=256 << 10))
    ck.declare_derived([(2 * k, 2 * k + 1) for k in range(len(counts))])
    ck.register_tensors(shard.descs())
    it = 0

    def snapshot():
        nonlocal it
        it += 1
        ck.snapshot_async(it, stream.cuda_stream)
        ck.wait_immutable_window_end(stream.cuda_stream)
        ck.flush(it)
        return ck.stats(it)["format_version"]

    assert snapshot() == 2
    whole = [gu.download(f) for f in shard.flat]
    good = ck.file_name(it)
    for k, n in enumerate(counts):
        p = bits[k][0]
        for e in sorted({0, n - 1, n // 4 * 4 - 1, min(n - 1, n // 4 * 4), min(n, 4096) - 1, min(n - 1, 4096), min(n, 8192) - 1, min(n - 1, 8192)}):
            if e < 0:
                continue
            wrong = np.array([p[e] ^ 1], dtype=np.uint16)
            B.proxy_copy_h2d(shard.ptrs[2 * k] + 2 * e, wrong.ctypes.data, 2)
            assert snapshot() == 1, (k, n, e)
            B.proxy_copy_h2d(shard.ptrs[2 * k] + 2 * e, p[e:e + 1].ctypes.data, 2)
    assert snapshot() == 2
    for k, n in enumerate(counts):      # the stored state stays, the derived one is lost; the guards keep their bytes
        junk = np.full(n, 0xABCD, dtype=np.uint16)
        B.proxy_copy_h2d(shard.ptrs[2 * k], junk.ctypes.data, junk.nbytes)
        zeros = np.zeros(n, dtype=np.uint32)
        B.proxy_copy_h2d(shard.ptrs[2 * k + 1], zeros.ctypes.data, zeros.nbytes)
    ck.restore(good, stream.cuda_stream)
    stream.synchronize()
    for f, w in zip(shard.flat, whole):
        assert np.array_equal(gu.download(f), w)
    ck.destroy()
    shard.free()
