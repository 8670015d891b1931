// A batch of tensor descriptors small enough to travel in a kernel's arguments (under 4 KiB).
#pragma once
#include <cstdint>

#if defined(__HIPCC__)
#define DSLLM_HOST_DEVICE __host__ __device__
#else
#define DSLLM_HOST_DEVICE
#endif

namespace dsllm {

// What pack_batch_kernel works through: pieces of tensors, in image order, compact so that many fit the kernel arguments
// (12 bytes each). Every piece fills whole 4 KiB pages of the image; all but a tensor's last piece are multiples of 4 KiB.
constexpr int kPackBatch = 320;
constexpr uint64_t kPackPage = 4096;                  // the file format's alignment unit
#ifndef DSLLM_PACK_BATCH_PAGES
#define DSLLM_PACK_BATCH_PAGES (1u << 23)             // 32 GiB of image per launch: a grid has fewer than 2^32 work-items
#endif
constexpr uint32_t kPackBatchPages = DSLLM_PACK_BATCH_PAGES;

struct PackBatch {
    uint64_t src_pad[kPackBatch];          // address of the piece's first byte (48 bits), zero bytes behind its last one << 48
    uint32_t first_page[kPackBatch + 1];   // page of the batch's image that the piece begins with; [count] = one past its last
    uint32_t count;

    DSLLM_HOST_DEVICE uint64_t src(uint32_t k) const { return src_pad[k] & 0xFFFFFFFFFFFFull; }
    DSLLM_HOST_DEVICE uint32_t pad(uint32_t k) const { return uint32_t(src_pad[k] >> 48); }
    DSLLM_HOST_DEVICE bool full() const { return count == uint32_t(kPackBatch) || first_page[count] == kPackBatchPages; }
    void clear() { count = 0; first_page[0] = 0; }
    // Takes as much of [addr, addr + nbytes) as there is room for (at least one page unless full()); returns the bytes taken.
    uint64_t add(uint64_t addr, uint64_t nbytes) {
        const uint64_t room = kPackBatchPages - first_page[count];
        uint64_t pages = (nbytes + kPackPage - 1) / kPackPage;
        uint64_t taken = nbytes;
        if (pages > room) { pages = room; taken = room * kPackPage; }
        src_pad[count] = addr | ((pages * kPackPage - taken) << 48);
        first_page[count + 1] = first_page[count] + uint32_t(pages);
        count++;
        return taken;
    }
};
static_assert(sizeof(PackBatch) <= 4000, "must fit the kernel argument segment with room to spare");

// tiles the padded extent of a tensor at data-region offset d0 is cut into (cuts at its start and at every multiple of tile_bytes)
inline uint64_t tiles_of(uint64_t d0, uint64_t nbytes, uint64_t tile_bytes) {
    const uint64_t dend = d0 + (nbytes + 4095) / 4096 * 4096;
    return (dend + tile_bytes - 1) / tile_bytes - d0 / tile_bytes;
}

}  // namespace dsllm
