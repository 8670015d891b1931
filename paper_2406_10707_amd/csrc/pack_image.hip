// ckpt_pack_image: the pack step on its own. A list of tensors is gathered into the image of its
// checkpoint data region in device memory, without a context: no ring, no threads, no file. The descriptors travel in
// kernel arguments, so neither entry point allocates or shares anything; ckpt_pack_image_noalloc is the one that does
// not wait for the stream.
#include "engine_internal.hpp"
#include "tile_batch.hpp"

// The largest list ckpt_pack_image_noalloc takes, in tiles of 32 KiB: its callers rely on what it refuses, and it bounds what
// the call enqueues without waiting to 103 launches.
constexpr uint64_t kNoallocTiles = 131072;

namespace dsllm {
hipError_t launch_pack_batch(PackBatch &bt, void *image, hipStream_t stream);
hipError_t launch_pack_batch(LongPackBatch &bt, void *image, hipStream_t stream);
}

using namespace dsllm;

namespace {

// Lists of more than kPackBatch tensors go in batches of four times as many with 15.5 KB of arguments: every launch
// less is some 2 us on the card and up to 5 on the host, and the longer arguments cost 0.1 (320 tensors 9.0 us, 324 9.1). Launches of 320 -> of 1280: 360 tensors
// 11.6 -> 8.8 us, 592 of 1 MB 12.3 -> 9.5, of 1.74 GB 523 -> 518, 2400 misaligned of 4.3 GB 1378 -> 1365, 16,000 of 5 MB 236 -> 101, of 213 MB
// 311 -> 188. Large tensors go in launches of 320: those take hundreds of microseconds, and a long sweep in runs is slower by more than a
// launch. Most of the bytes off the 128-byte lines: 3000 tensors of 1.5 MiB 1481 -> 1480, 1200 of 2 MiB 795 -> 801, of 3 MiB 1180 -> 1195, of 5 MiB 1958 -> 1988,
// 400 of 17 MiB 2223 -> 2243. On them: 1200 of 3 MiB 1122 -> 1117, of 5 MiB 1847 -> 1840, of 7 MiB 2576 -> 2573, 400 of 9 MiB 1114 -> 1119, of 17 MiB
// 2084 -> 2094.
constexpr uint64_t kLongMean = 8ull << 20, kLongMeanOffLines = 2ull << 20;

// What both entry points check before anything is launched: every tensor is device memory of the
// current GPU and lies inside its allocation, the destination is device memory of the same GPU, 16-byte
// aligned and large enough. Returns the number of tiles and whether the list goes in long launches.
int check_pack_arguments(const ckpt_tensor_desc *tensors, size_t n, const void *dev_dst, uint64_t dst_bytes, uint64_t *n_tiles_out, bool *long_launches) {
    if (!tensors || n == 0 || !dev_dst) return fail(CKPT_EINVAL, "null argument or empty tensor list");
    int dev = 0;
    HIP_TRY(nullptr, hipGetDevice(&dev));
    // The allocations the list has touched so far, the latest eight of them: tensors mostly share a few (flat buffers, an
    // allocator's segments), and what the runtime says of one address of an allocation it says of all of them. Two
    // queries per tensor were 0.12 us each: 13 of the 24 us the host spent on 112 tensors, 0.3 of 2.05 ms on 2400.
    struct Span { uint64_t lo, hi; } spans[8];
    uint32_t held = 0, recent = 0, oldest = 0;      // how many, the one found last, the one to be replaced once all eight are in use
    // 0: fine; 1: not device memory of this GPU; 2: runs past its allocation (queries only, nothing is allocated;
    // texts are put together on the failing path alone)
    auto on_this_gpu = [&](const void *p, uint64_t nbytes) -> int {
        const uint64_t a = uint64_t(p);
        for (uint32_t i = 0, j = recent; i < held; i++, j = j + 1 < held ? j + 1 : 0)
            if (a >= spans[j].lo && a < spans[j].hi) { recent = j; return nbytes > spans[j].hi - a ? 2 : 0; }
        hipPointerAttribute_t attr;
        hipError_t e = hipPointerGetAttributes(&attr, p);
        if (e != hipSuccess || attr.type != hipMemoryTypeDevice || attr.device != dev) { (void)hipGetLastError(); return 1; }
        void *base = nullptr; size_t span = 0;
        e = hipMemGetAddressRange(reinterpret_cast<hipDeviceptr_t *>(&base), &span, reinterpret_cast<hipDeviceptr_t>(const_cast<void *>(p)));
        if (e != hipSuccess) { (void)hipGetLastError(); return 0; }
        if (held < 8) recent = held++;
        else { recent = oldest; oldest = (oldest + 1) % 8; }
        spans[recent] = Span{uint64_t(base), uint64_t(base) + span};
        return nbytes > uint64_t(base) + span - a ? 2 : 0;
    };
    static const char *const why[] = {"", ": not device memory of the current GPU", ": range runs past its allocation"};
    uint64_t off = 0, tiles = 0;
    for (size_t k = 0; k < n; k++) {
        const ckpt_tensor_desc &d = tensors[k];
        if (d.dtype & CKPT_PLACE_HOST) return fail(CKPT_EINVAL, "tensor " + std::to_string(k) + ": host-resident objects cannot be packed on the device");
        if (!d.dev_ptr || d.nbytes == 0) return fail(CKPT_EINVAL, "tensor " + std::to_string(k) + ": null pointer or zero bytes");
        if (int bad = on_this_gpu(d.dev_ptr, d.nbytes)) return fail(CKPT_EINVAL, "tensor " + std::to_string(k) + why[bad]);
        tiles += tiles_of(off, d.nbytes, kTileBytes);
        off += (d.nbytes + kAlign - 1) / kAlign * kAlign;
    }
    if (uint64_t(dev_dst) % 16 != 0) return fail(CKPT_EINVAL, "destination must be 16-byte aligned");
    if (dst_bytes < off) return fail(CKPT_EINVAL, "destination smaller than the data region (" + std::to_string(off) + " bytes)");
    if (int bad = on_this_gpu(dev_dst, off)) return fail(CKPT_EINVAL, std::string("destination") + why[bad]);
    if (tiles > 0xFFFFFFFFull) return fail(CKPT_EINVAL, "more than 2^32 tiles");
    *n_tiles_out = tiles;
    *long_launches = n > size_t(kPackBatch) && off / n <= kLongMean;
    if (*long_launches && off / n > kLongMeanOffLines) {
        uint64_t off_lines = 0;
        for (size_t k = 0; k < n; k++)
            if (uint64_t(tensors[k].dev_ptr) % 128) off_lines += tensors[k].nbytes;
        *long_launches = off_lines <= off / 2;
    }
    return CKPT_OK;
}

// Enqueues, on `stream`, the kernels that write the image: one for every batch of tensors. Allocates nothing, on either side.
template <class Batch>
int enqueue_batches(const ckpt_tensor_desc *tensors, size_t n, void *dev_dst, hipStream_t stream) {
    Batch bt;
    bt.clear();
    uint8_t *image = static_cast<uint8_t *>(dev_dst);
    auto launch = [&]() -> int {
        HIP_TRY(nullptr, launch_pack_batch(bt, image, stream));
        image += kPackPage * bt.pages;
        bt.clear();
        return CKPT_OK;
    };
    for (size_t k = 0; k < n; k++) {
        uint64_t addr = uint64_t(tensors[k].dev_ptr), left = tensors[k].nbytes;
        while (left) {
            const uint64_t taken = bt.add(addr, left);
            addr += taken;
            left -= taken;
            if (bt.full())
                if (int r = launch()) return r;
        }
    }
    return bt.count ? launch() : CKPT_OK;
}
int enqueue_pack_image(const ckpt_tensor_desc *tensors, size_t n, bool long_launches, void *dev_dst, hipStream_t stream) {
    return long_launches ? enqueue_batches<LongPackBatch>(tensors, n, dev_dst, stream) : enqueue_batches<PackBatch>(tensors, n, dev_dst, stream);
}

}  // namespace

// Called by ckpt_init for its device, so that a caller who has a context never meets the first launch of these kernels
// (which loads their code) inside a region where nothing may be allocated.
int dsllm::pack_image_setup(hipStream_t stream) {
    LongPackBatch bt;
    bt.clear();
    HIP_TRY(nullptr, launch_pack_batch(bt, nullptr, stream));
    return CKPT_OK;
}

extern "C" {

int ckpt_pack_image_noalloc(const ckpt_tensor_desc *tensors, size_t n, void *dev_dst, uint64_t dst_bytes, void *hip_stream) {
    uint64_t n_tiles = 0;
    bool long_launches = false;
    int r = check_pack_arguments(tensors, n, dev_dst, dst_bytes, &n_tiles, &long_launches);
    if (r) return r;
    if (n_tiles > kNoallocTiles)
        return fail(CKPT_EINVAL, "tensor list needs " + std::to_string(n_tiles) + " tiles, this entry point takes " + std::to_string(kNoallocTiles) +
                                     " (about 4 GiB of data region): use ckpt_pack_image");
    return enqueue_pack_image(tensors, n, long_launches, dev_dst, static_cast<hipStream_t>(hip_stream));
}

int ckpt_pack_image(const ckpt_tensor_desc *tensors, size_t n, void *dev_dst, uint64_t dst_bytes, void *hip_stream) {
    uint64_t n_tiles = 0;
    bool long_launches = false;
    int r = check_pack_arguments(tensors, n, dev_dst, dst_bytes, &n_tiles, &long_launches);
    if (r) return r;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    r = enqueue_pack_image(tensors, n, long_launches, dev_dst, stream);
    hipError_t es = hipStreamSynchronize(stream);
    if (r) return r;
    if (es != hipSuccess) return fail(CKPT_EHIP, std::string("hipStreamSynchronize: ") + hipGetErrorString(es));
    return CKPT_OK;
}

}  // extern "C"
