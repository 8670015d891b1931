"""Run as a program by tests/test_gpu_torch_interop.py (a process of its own: PyTorch has to be imported
before the library, so that the process holds one HIP runtime, PyTorch's).

PyTorch owns the device memory and the stream; the library gets raw pointers and the stream handle.
A few steps of a toy training loop with snapshots in between, files compared with the CPU oracle on
clones taken at each boundary, then a restore into overwritten tensors; and the pack entry point without allocation
in a captured graph, whose replays read the tensors as they are then."""
import sys
import tempfile

import torch  # noqa: E402  (first on purpose)

from oracle import oracle  # noqa: E402
from paper_2406_10707_amd import binding as B  # noqa: E402

DT = {torch.bfloat16: B.CKPT_BF16, torch.float32: B.CKPT_F32}


def as_bytes(t):
    return t.detach().contiguous().flatten().view(torch.uint8).cpu().numpy()


def captured_packs(dev, stream):
    """Lists whose descriptors fill the kernel arguments of each size (the largest 15.5 KB), one launch and several."""
    for n in (20, 100, 300, 1000, 1400):
        print(f"captured pack of {n} tensors", flush=True)
        arena = torch.randint(0, 256, (n * 5000,), dtype=torch.uint8, device=dev)
        sizes = [4096 * (k % 2) + 1 + 61 * k % 700 for k in range(n)]
        descs = [(f"t{k}", B.CKPT_U8, (b,), arena.data_ptr() + 5000 * k + k % 3, b) for k, b in enumerate(sizes)]
        data = sum(-(-b // 4096) * 4096 for b in sizes)
        image, eager = (torch.full((data,), 0xEE, dtype=torch.uint8, device=dev) for _ in range(2))
        graph = torch.cuda.CUDAGraph()
        stream.synchronize()
        with torch.cuda.graph(graph, stream=stream):
            B.pack_image_noalloc(descs, image.data_ptr(), data, stream.cuda_stream)
        with torch.cuda.stream(stream):
            for replay in range(4):
                arena.add_(replay + 1)
                image.fill_(0xEE)
                B.pack_image_noalloc(descs, eager.data_ptr(), data, stream.cuda_stream)
                graph.replay()
                stream.synchronize()
                assert torch.equal(image, eager), f"replay {replay}"
                host, off = as_bytes(image), 0
                src = as_bytes(arena)
                for k, b in enumerate(sizes):
                    assert (host[off:off + b] == src[5000 * k + k % 3:5000 * k + k % 3 + b]).all(), (replay, k)
                    off += -(-b // 4096) * 4096


def main():
    dev = torch.device("cuda:0")
    torch.manual_seed(7)
    shapes = [(513, 257), (1000,), (64, 64, 33), (3,), (2048, 1024)]
    state, names = [], []
    for k, shp in enumerate(shapes):
        master = (torch.randn(*shp) * 0.02).to(dev)
        for role, t in (("p_bf16", master.to(torch.bfloat16)), ("master", master), ("m", torch.zeros_like(master)),
                        ("v", torch.zeros_like(master))):
            state.append(t)
            names.append(f"param{k}.{role}")
    descs = [(n, DT[t.dtype], tuple(t.shape), t.data_ptr(), t.numel() * t.element_size()) for n, t in zip(names, state)]
    out_dir = tempfile.mkdtemp(prefix="dsllm_torch_")
    ck = B.Checkpointer(B.make_config(out_dir=out_dir, dma_chunk_bytes=256 << 10, pack_superchunk_bytes=1 << 20, host_ring_bytes=2 << 20))
    ck.register_tensors(descs)
    stream = torch.cuda.Stream()
    a = torch.randn(1024, 1024, device=dev)
    clones = {}
    with torch.cuda.stream(stream):
        for it in range(1, 5):
            b = a @ a                                            # forward/backward stand-in on the same stream
            ck.wait_immutable_window_end(stream.cuda_stream)     # before anything mutates the state
            for k in range(len(shapes)):
                p, master, m, v = state[4 * k:4 * k + 4]
                grad = torch.full_like(master, 1e-3 * it)
                m.mul_(0.9).add_(grad, alpha=0.1)
                v.mul_(0.999).addcmul_(grad, grad, value=0.001)
                master.addcdiv_(m, v.sqrt() + 1e-8, value=-1e-3)
                p.copy_(master)
            clones[it] = [t.clone() for t in state]
            ck.snapshot_async(it, stream.cuda_stream)
            del b
    ck.flush()
    stream.synchronize()
    for it in range(1, 5):
        tensors = [(n, DT[t.dtype], tuple(t.shape), as_bytes(c)) for n, t, c in zip(names, state, clones[it])]
        bad = oracle.compare_file(tensors, it, ck.file_name(it))
        assert bad is None, f"iteration {it}: {bad}"
    with torch.cuda.stream(stream):
        for t in state:
            t.fill_(7.0)
        assert ck.restore(ck.file_name(2), stream.cuda_stream) == 2
    stream.synchronize()
    for t, c in zip(state, clones[2]):
        assert torch.equal(t, c)
    captured_packs(dev, stream)
    ck.destroy()
    print("torch interop ok:", torch.__version__, "hip", torch.version.hip, flush=True)


if __name__ == "__main__":
    sys.exit(main())
