// A batch of tensor descriptors small enough to travel in a kernel's arguments (under 4 KiB, of long lists under 16).
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
constexpr int kPackBatch = 320, kLongPackBatch = 1280;      // pieces of a launch; of a launch of a list of more than kPackBatch tensors
constexpr uint64_t kPackPage = 4096;                  // the file format's alignment unit
#ifndef DSLLM_PACK_BATCH_PAGES
#define DSLLM_PACK_BATCH_PAGES (1u << 23)             // 32 GiB of image per launch: a grid has fewer than 2^32 work-items
#endif
constexpr uint32_t kPackBatchPages = DSLLM_PACK_BATCH_PAGES;

// A list of up to N pieces as a kernel's argument. A page's piece is between the first and the last one of its group of
// 2^group_bits pages, where bisection finds it; with large tensors they are mostly the same.
constexpr uint32_t pack_groups(int pieces) { return pieces > kPackBatch ? 128 : 32; }
struct PackSource { uint64_t src; uint32_t bytes; };       // a page's first byte, how many of its 4 KiB are the tensor's
template <int N>
struct PackArgs {
    uint32_t pages, group_bits;
    uint32_t group[pack_groups(N)];        // first piece of the group's pages, last piece << 16
    uint64_t src_pad[N];                   // address of the piece's first byte (48 bits), zero bytes behind its last one << 48
    uint32_t first_page[N + 1];            // page of the batch's image that the piece begins with; behind the last one: one past its last

    DSLLM_HOST_DEVICE PackSource of(uint32_t page) const {
        const uint32_t both = group[page >> group_bits];
        uint32_t lo = both & 0xFFFF, hi = both >> 16;
        while (lo < hi) {
            const uint32_t mid = (lo + hi + 1) / 2;
            if (first_page[mid] <= page) lo = mid;
            else hi = mid - 1;
        }
        const uint64_t from = src_pad[lo];
        const uint32_t first = first_page[lo], end = first_page[lo + 1];
        return PackSource{(from & 0xFFFFFFFFFFFFull) + kPackPage * (page - first), uint32_t(kPackPage) - (page + 1 == end ? uint32_t(from >> 48) : 0)};
    }
};
static_assert(sizeof(PackArgs<kPackBatch>) <= 4000 && sizeof(PackArgs<kLongPackBatch>) <= 16000, "must fit the kernel argument segment with room to spare");

template <int MOST>
struct PackBatchOf : PackArgs<MOST> {
    using PackArgs<MOST>::pages;
    using PackArgs<MOST>::group_bits;
    using PackArgs<MOST>::group;
    using PackArgs<MOST>::src_pad;
    using PackArgs<MOST>::first_page;
    uint32_t count;

    uint64_t src(uint32_t k) const { return src_pad[k] & 0xFFFFFFFFFFFFull; }
    uint32_t pad(uint32_t k) const { return uint32_t(src_pad[k] >> 48); }
    bool full() const { return count == uint32_t(MOST) || pages == kPackBatchPages; }
    void clear() { count = 0; pages = first_page[0] = 0; }
    // Takes as much of [addr, addr + nbytes) as there is room for (at least one page unless full()); returns the bytes taken.
    uint64_t add(uint64_t addr, uint64_t nbytes) {
        const uint64_t room = kPackBatchPages - pages;
        uint64_t n = (nbytes + kPackPage - 1) / kPackPage;
        uint64_t taken = nbytes;
        if (n > room) { n = room; taken = room * kPackPage; }
        src_pad[count] = addr | ((n * kPackPage - taken) << 48);
        pages = first_page[++count] = pages + uint32_t(n);
        return taken;
    }
    // One group where groups don't pay.
    void make_groups(bool pay) {
        group_bits = 31;
        group[0] = (count ? count - 1 : 0) << 16;
        if (!pay || !count) return;
        const uint32_t groups = pack_groups(int(count));      // those of the shortest arguments that hold the list
        for (group_bits = 0; (pages - 1) >> group_bits >= groups;) group_bits++;
        uint32_t k = 0;
        for (uint32_t g = 0; uint64_t(g) << group_bits < pages; g++) {
            const uint64_t begin = uint64_t(g) << group_bits, end = begin + (1ull << group_bits);
            while (first_page[k + 1] <= begin) k++;
            group[g] = k;
            while (k + 1 < count && first_page[k + 1] < end) k++;
            group[g] |= k << 16;
        }
    }
    template <int N>
    PackArgs<N> shorter() const {          // count is at most N
        if constexpr (N == MOST) return *this;
        PackArgs<N> a;
        a.pages = pages;
        a.group_bits = group_bits;
        for (uint32_t g = 0; g < pack_groups(N); g++) a.group[g] = group[g];
        for (uint32_t k = 0; k < count; k++) { a.src_pad[k] = src_pad[k]; a.first_page[k] = first_page[k]; }
        a.first_page[count] = pages;
        return a;
    }
};
typedef PackBatchOf<kPackBatch> PackBatch;
typedef PackBatchOf<kLongPackBatch> LongPackBatch;

// tiles the padded extent of a tensor at data-region offset d0 is cut into (cuts at its start and at every multiple of tile_bytes)
inline uint64_t tiles_of(uint64_t d0, uint64_t nbytes, uint64_t tile_bytes) {
    const uint64_t dend = d0 + (nbytes + 4095) / 4096 * 4096;
    return (dend + tile_bytes - 1) / tile_bytes - d0 / tile_bytes;
}

}  // namespace dsllm
