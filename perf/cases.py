"""The calls whose speed this repository answers for: the pack step on its own, whole snapshots, restores, and the two
kernels of the training proxy that stands in for the job being checkpointed (include/ckpt.h, include/ckpt_proxy.h).

Byte movers are compared bit for bit. A shard is built the way the repository's workloads are (shards.py): every
parameter has four state tensors, a bf16 working copy, f32 master weights and two f32 Adam moments, which lie in one
arena per role. With `pad` the tensors start at multiples of 128 elements, as allocations of their own do; without it
they follow each other with gaps of a few elements, as in flattened optimizer buffers, so that most starts are aligned
to the element size only.
"""
import math
import os
import random
import tempfile

import numpy as np
import torch

from paper_2406_10707_amd import binding as B
from paper_2406_10707_amd import shards

ROLES = (("p_bf16", torch.bfloat16, 2, B.CKPT_BF16), ("master", torch.float32, 4, B.CKPT_F32),
         ("m", torch.float32, 4, B.CKPT_F32), ("v", torch.float32, 4, B.CKPT_F32))
UNIT = 4096          # alignment of a tensor in the data region (docs/FORMAT.md)
MIB = 1 << 20
ADAM = {"lr": 1e-3, "beta1": 0.9, "beta2": 0.999, "eps": 1e-8}


# ------------------------------------------------------------------ the cases

def listed():
    return [
        # The smallest call: the structure of a small model's whole state (112 tensors, 0.4 MB of payload), packed in place
        # by a caller that may not allocate. Latency, launches and host work per tensor.
        dict(name="pack-tiny", kind="pack", entry="noalloc", shard="gpt2", layers=2, hidden=24, vocab=503, pad=1),
        # The state of a 124 M parameter model in 592 tensors, 1.74 GB: the ordinary call, same entry point.
        dict(name="pack-gpt2", kind="pack", entry="noalloc", shard="gpt2", layers=12, hidden=768, vocab=50257, pad=1),
        # Flattened optimizer buffers: 2400 ragged fragments at element-aligned addresses, about 4 GB.
        dict(name="pack-fragments", kind="pack", entry="image", shard="fragments", params=600, lo=1000, hi=4000000, pad=0),
        # The largest: four layers of a 7B model, few and large tensors, 11 GB.
        dict(name="pack-llama", kind="pack", entry="image", shard="llama", layers=4, hidden=4096, ffn=11008, heads=32, kv=32, tp=1, pad=1),
        # A checkpoint of a very small state, as in fine-tuning a few parameters: request to committed file. Latency.
        dict(name="snapshot-tiny", kind="snapshot", shard="gpt2", layers=2, hidden=24, vocab=503, pad=1, reduce=0, direct=0, chunk=64 * MIB),
        # The ordinary checkpoint: 1.74 GB, request to committed file.
        dict(name="snapshot-gpt2", kind="snapshot", shard="gpt2", layers=12, hidden=768, vocab=50257, pad=1, reduce=0, direct=0, chunk=64 * MIB),
        # Data reduction on flattened buffers: every bf16 copy is checked against its f32 source on the device and left out.
        dict(name="snapshot-reduced", kind="snapshot", shard="fragments", params=120, lo=1000, hi=4000000, pad=0, reduce=1, direct=0, chunk=64 * MIB),
        # Restart of a small job: one layer of the 124 M parameter model with its optimizer state, 0.1 GB.
        dict(name="restore-small", kind="restore", shard="gpt2", layers=1, hidden=768, vocab=503, pad=1, reduce=0, direct=0, chunk=64 * MIB),
        # Restart from a reduced file into flattened buffers: scatter to unaligned addresses, bf16 copies recomputed.
        dict(name="restore-reduced", kind="restore", shard="fragments", params=120, lo=1000, hi=4000000, pad=0, reduce=1, direct=0, chunk=64 * MIB),
        # The update phase of the training proxy: the nine parameters of a 7B model's layer, 202 M elements.
        dict(name="adam-llama-layer", kind="adam", shard="llama", layers=1, hidden=4096, ffn=11008, heads=32, kv=32, tp=1, pad=1),
        # The forward and backward stand-in of the training proxy, in the size that the benchmark runs.
        dict(name="gemm-8192", kind="gemm", m=8192, n=8192, k=8192),
        # The same for a small model: 1024 tokens through the first product of a 768-wide MLP. Few tiles, short K.
        dict(name="gemm-1024x3072x768", kind="gemm", m=1024, n=3072, k=768),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_shard(rng, most_elements):
    """Shard of a random layout with at most `most_elements` parameters, sizes spread over the logarithm of the range."""
    what = rng.choice(("gpt2", "llama", "fragments"))
    target = _log(rng, 20000, most_elements)
    if what == "fragments":
        lo = _log(rng, 1, 5000)
        hi = _log(rng, 4 * lo, 4 * MIB)
        mean = (hi - lo) / math.log(hi / lo)
        return dict(shard=what, params=max(1, min(4000, int(target / mean))), lo=lo, hi=min(hi, most_elements), pad=rng.randint(0, 1))
    layers = rng.randint(1, 12)
    if what == "gpt2":        # 12 hidden^2 elements a layer
        hidden = max(24, 8 * int(math.sqrt(target / (12 * layers)) / 8))
        vocab = max(1, min(50257, int(target / (4 * hidden))))
        return dict(shard=what, layers=layers, hidden=hidden, vocab=vocab, pad=rng.randint(0, 1))
    heads = rng.choice((4, 8, 32))
    kv = rng.choice((heads, 4))
    tp = rng.choice((1, 2, 4))
    unit = heads * 4
    hidden = max(unit, unit * int(math.sqrt(tp * target / (12 * layers)) / unit))
    return dict(shard=what, layers=layers, hidden=hidden, ffn=tp * (hidden * 43 // (16 * tp)), heads=heads, kv=kv, tp=tp, pad=rng.randint(0, 1))


def draw(rng):
    kind = rng.choice(("pack", "pack", "pack", "snapshot", "snapshot", "restore", "restore", "adam", "gemm", "gemm"))
    if kind == "gemm":
        return dict(kind=kind, m=128 * _log(rng, 1, 64), n=128 * _log(rng, 1, 64), k=64 * _log(rng, 1, 128))
    if kind == "adam":
        c = dict(kind=kind, **_draw_shard(rng, 200_000_000))
        c["pad"] = 1          # the update needs 16-byte aligned tensors
        return c
    if kind == "pack":
        c = _draw_shard(rng, 600_000_000)
        small = sum(math.prod(s) for s in _shapes(c)) < 200_000_000      # the table of the entry point without allocation ends at about 4 GiB
        return dict(kind=kind, entry=rng.choice(("noalloc", "image")) if small else "image", **c)
    return dict(kind=kind, **_draw_shard(rng, 120_000_000), reduce=rng.randint(0, 1), direct=rng.choice((0, 0, 16 * MIB)),
                chunk=rng.choice((64 * MIB, 64 * MIB, 256 * MIB)))


# ------------------------------------------------------------------ shards

def _shapes(case):
    if case["shard"] == "gpt2":
        return [s for _, s in shards.gpt2_params(vocab=case["vocab"], hidden=case["hidden"], layers=case["layers"], npos=max(32, case["hidden"]))]
    if case["shard"] == "llama":
        return [s for _, s in shards.llama_params(case["layers"], case["hidden"], case["ffn"], 1, case["heads"], case["kv"], tp=case["tp"],
                                                  first_stage=False, last_stage=False)]
    r = random.Random("%(params)d %(lo)d %(hi)d" % case)
    return [(max(1, _log(r, case["lo"], case["hi"])),) for _ in range(case["params"])]


def _layout(case):
    """Element offset of every parameter in the arenas, and the arenas' length in elements."""
    r = random.Random(len(_shapes(case)))
    offs, at = [], 0
    for s in _shapes(case):
        at = -(-at // 128) * 128 if case["pad"] else at + r.randint(0, 15)
        offs.append(at)
        at += math.prod(s)
    return offs, -(-at // 128) * 128


def _payload(case):
    return sum(14 * math.prod(s) for s in _shapes(case))


def _data_bytes(case, reduced=False):
    return sum(-(-es * math.prod(s) // UNIT) * UNIT for s in _shapes(case) for role, _, es, _ in ROLES if not (reduced and role == "p_bf16"))


def _arenas(case, seed):
    """One tensor per role: master and m ~ N(0, 0.02), the bf16 copy the rounding of master, v = N(0, 1e-3)^2."""
    n = _layout(case)[1]
    g = torch.Generator(device="cuda").manual_seed(seed)
    master = torch.randn(n, device="cuda", generator=g).mul_(0.02)
    m = torch.randn(n, device="cuda", generator=g).mul_(0.02)
    v = torch.randn(n, device="cuda", generator=g).mul_(1e-3).square_()
    return {"p_bf16": master.to(torch.bfloat16), "master": master, "m": m, "v": v}


def _tensors(case, arenas):
    out = []
    for k, (shape, off) in enumerate(zip(_shapes(case), _layout(case)[0])):
        for role, _, es, code in ROLES:
            out.append(("param%d.%s" % (k, role), code, shape, arenas[role].data_ptr() + es * off, es * math.prod(shape)))
    return out


def _stream():
    return torch.cuda.current_stream().cuda_stream


def _engine(case, tensors, out_dir):
    """A context as a training loop on a memory file system makes it: pinned ring for the shard (1 GiB at most), files recycled in place."""
    ring = min(1 << 30, -(-_data_bytes(case) // case["chunk"]) * case["chunk"])
    ck = B.Checkpointer(B.make_config(out_dir=out_dir, host_ring_bytes=ring, dma_chunk_bytes=case["chunk"], keep_last=1, prealloc_files=2,
                                      pack_superchunk_bytes=1 << 30, direct_min_bytes=case["direct"]))
    if case["reduce"]:
        ck.declare_derived([(4 * k, 4 * k + 1) for k in range(len(tensors) // 4)])
    ck.register_tensors(tensors)
    return ck


# ------------------------------------------------------------------ one pass

def prepare(case, seed):
    if case["kind"] == "gemm":
        g = torch.Generator(device="cuda").manual_seed(seed)
        a = torch.randn(case["m"], case["k"], device="cuda", generator=g).mul_(0.05).to(torch.bfloat16)
        b = torch.randn(case["n"], case["k"], device="cuda", generator=g).mul_(0.05).to(torch.bfloat16)
        return {"case": case, "a": a, "b": b, "c": torch.empty(case["m"], case["n"], device="cuda", dtype=torch.bfloat16)}
    arenas = _arenas(case, seed)
    tensors = _tensors(case, arenas)
    s = {"case": case, "arenas": arenas}
    if case["kind"] == "adam":
        s["params"] = [[t[3] for t in tensors[k:k + 4]] + [math.prod(tensors[k][2])] for k in range(0, len(tensors), 4)]
        s["seed"], s["step"] = seed, 0
    elif case["kind"] == "pack":
        # a program that packs again and again keeps its descriptor array
        s["descs"], s["keep"] = B.make_descs(tensors)
        s["n"] = len(tensors)
        s["image"] = torch.empty(_data_bytes(case) // 8, device="cuda", dtype=torch.int64)
    else:
        s["dir"] = tempfile.TemporaryDirectory(prefix="dsllm_cases_", dir="/dev/shm" if os.path.isdir("/dev/shm") else None)
        s["ck"], s["it"] = _engine(case, tensors, s["dir"].name), 0
        if case["kind"] == "restore":      # a file to come back to, then the state of a program that has just started
            s["ck"].snapshot_async(1, _stream())
            s["ck"].wait_immutable_window_end(_stream())
            s["ck"].flush(1)
            s["path"] = s["ck"].file_name(1)
            for t in arenas.values():
                t.zero_()
    torch.cuda.synchronize()
    return s


def run(s):
    kind = s["case"]["kind"]
    if kind == "pack":
        call = B.lib.ckpt_pack_image_noalloc if s["case"]["entry"] == "noalloc" else B.lib.ckpt_pack_image
        rc = call(s["descs"], s["n"], s["image"].data_ptr(), 8 * s["image"].numel(), _stream())
        if rc != 0:
            raise RuntimeError(B.lib.ckpt_last_error().decode())
        return s["image"]
    if kind == "snapshot":
        s["it"] += 1
        s["ck"].snapshot_async(s["it"], _stream())
        s["ck"].wait_immutable_window_end(_stream())
        s["ck"].flush(s["it"])
        whole = np.memmap(s["ck"].file_name(s["it"]), dtype=np.int64, mode="r")
        return whole
    if kind == "restore":
        s["ck"].restore(s["path"], _stream())
        return [t.view(torch.int16) if t.dtype == torch.bfloat16 else t.view(torch.int32) for t in s["arenas"].values()]
    if kind == "adam":
        s["step"] += 1
        st = _stream()
        for k, (p, w, m, v, n) in enumerate(s["params"]):
            B.proxy_adam_step(p, w, m, v, n, s["seed"], k, s["step"], st, **ADAM)
        return s["arenas"]
    B.proxy_gemm_bf16(s["a"].data_ptr(), s["b"].data_ptr(), s["c"].data_ptr(), s["case"]["m"], s["case"]["n"], s["case"]["k"], _stream())
    return s["c"]


# ------------------------------------------------------------------ what a pass cannot do without

def work(case):
    if case["kind"] == "gemm":
        m, n, k = case["m"], case["n"], case["k"]
        return {"bytes": 2 * (m * k + n * k + m * n), "flops": 2 * m * n * k}
    if case["kind"] == "adam":      # four tensors read, four written
        return {"bytes": 2 * _payload(case), "flops": 0}
    if case["kind"] == "pack":
        return {"bytes": _payload(case) + _data_bytes(case), "flops": 0}
    if case["kind"] == "snapshot":  # the state read (a derived copy too: it is checked), the file written
        return {"bytes": _payload(case) + _data_bytes(case, case["reduce"]), "flops": 0}
    return {"bytes": _data_bytes(case, case["reduce"]) + _payload(case), "flops": 0}      # the file read, the state written


def tolerance(case):
    if case["kind"] == "gemm":
        # f32 sums in another order move a result across a rounding boundary of bf16 now and then, by at most 2^-7 of the
        # value: against the rounded 64-bit product 4.8e-5 (rel) at K = 8192, and two such paths may part on both sides
        return {"rel": 2e-4, "max": 1.6e-2}
    if case["kind"] == "adam":
        # f32 arithmetic with other roundings: 7e-8 of the f32 tensors; the bf16 copy rounds to the other side now and then:
        # 9.5e-6 against the rounded 64-bit result
        return {"rel": 4e-5, "max": 1.6e-2}
    return "exact"


# ------------------------------------------------------------------ the same in 64 bits

def _mix(x):
    """The counter-based generator of include/ckpt_proxy.h on int64 tensors (wrapping products, logical shifts)."""
    def signed(u):
        return u - (1 << 64) if u >= 1 << 63 else u

    def shr(v, s):
        return (v >> s) & ((1 << (64 - s)) - 1)

    z = x + signed(0x9E3779B97F4A7C15)
    z = (z ^ shr(z, 30)) * signed(0xBF58476D1CE4E5B9)
    z = (z ^ shr(z, 27)) * signed(0x94D049BB133111EB)
    return z ^ shr(z, 31)


def _mix_one(x):
    return int(_mix(torch.tensor([x - (1 << 64) if x >= 1 << 63 else x], dtype=torch.int64))[0]) & ((1 << 64) - 1)


def exact(case, seed):
    if case["kind"] == "gemm":
        s = prepare(case, seed)
        return s["a"].double() @ s["b"].double().t()
    if case["kind"] != "adam":
        return None
    a = _arenas(case, seed)
    f32 = lambda x: float(np.float32(x))  # noqa: E731  the constants arrive in f32
    lr, b1, b2, eps = (f32(ADAM[k]) for k in ("lr", "beta1", "beta2", "eps"))
    out = {k: t.double() for k, t in a.items()}
    for k, (shape, off) in enumerate(zip(_shapes(case), _layout(case)[0])):
        n = math.prod(shape)
        at = slice(off, off + n)
        key = _mix_one((seed + 1) ^ _mix_one(4 * k + 3))
        r = _mix(torch.arange(n, device="cuda", dtype=torch.int64))
        r = _mix(r ^ (key - (1 << 64) if key >= 1 << 63 else key))
        g = 0.001 * (2.0 * (((r >> 40) & 0xFFFFFF).double() / (1 << 24)) - 1.0)
        del r
        m = b1 * out["m"][at] + (1.0 - b1) * g
        v = b2 * out["v"][at] + (1.0 - b2) * g * g
        w = out["master"][at] - lr * (m / (1.0 - b1)) / ((v / (1.0 - b2)).sqrt() + eps)
        out["m"][at], out["v"][at], out["master"][at], out["p_bf16"][at] = m, v, w, w
    return out
