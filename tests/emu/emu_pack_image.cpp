// The entry points that pack a list of tensors, on the CPU model of the runtime (hip/hip_runtime.h) with a table of
// allocations: what is asked of the runtime about each list, what is refused, and the image. Meant for -fsanitize=address.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include <sys/uio.h>

#include "../../include/ckpt.h"
#include "hip/hip_runtime.h"

thread_local dim3 threadIdx, blockIdx, blockDim, gridDim;
ssize_t emu_pwrite(int, const void *, size_t, off_t) { return -1; }   // no file is written here
#define REQUIRE(x) do { if (!(x)) { printf("FAILED line %d: %s (%s)\n", __LINE__, #x, ckpt_last_error()); exit(1); } } while (0)

struct Allocation { uint8_t *base; size_t size; };
static std::vector<Allocation> g_allocations;
static bool allocation_of(const void *p, void **base, size_t *size) {
    for (auto &a : g_allocations)
        if (p >= a.base && p < a.base + a.size) { *base = a.base; *size = a.size; return true; }
    return false;
}

int main() {
    const uint64_t size = 64 << 10;
    for (int i = 0; i < 13; i++) g_allocations.push_back({static_cast<uint8_t *>(aligned_alloc(4096, i == 12 ? 4 << 20 : size)), i == 12 ? size_t(4 << 20) : size_t(size)});
    for (int i = 0; i < 12; i++) for (uint64_t j = 0; j < size; j++) g_allocations[i].base[j] = uint8_t(i * 41 + j * 7 + (j >> 8));
    g_emu_allocation_of = allocation_of;
    uint8_t *const image = g_allocations[12].base;

    // `arenas` allocations in turn, as a list of parameters with so many state tensors each visits them
    auto list = [&](int n, int arenas) {
        std::vector<ckpt_tensor_desc> d(n);
        for (int k = 0; k < n; k++) { d[k].dev_ptr = g_allocations[k % arenas].base + 100 * (k / arenas) + k % 16; d[k].nbytes = uint64_t(50 + k % 40); }
        return d;
    };
    for (auto pack : {ckpt_pack_image, ckpt_pack_image_noalloc})
        for (int arenas : {1, 2, 3, 4, 7, 8, 9, 12}) {
            auto d = list(120, arenas);
            memset(image, 0xCC, 4 << 20);
            g_emu_pointer_queries = 0;
            REQUIRE(pack(d.data(), d.size(), image, 4 << 20, nullptr) == CKPT_OK);
            // one query for each allocation and one for the destination, where the allocations in use are held
            if (arenas <= 8 && g_emu_pointer_queries != arenas + 1) { printf("FAILED %d allocations: %d queries\n", arenas, g_emu_pointer_queries.load()); return 1; }
            REQUIRE(g_emu_pointer_queries <= 121);
            for (size_t k = 0; k < d.size(); k++) {
                REQUIRE(memcmp(image + 4096 * k, d[k].dev_ptr, d[k].nbytes) == 0);
                for (uint64_t i = d[k].nbytes; i < 4096; i++) REQUIRE(image[4096 * k + i] == 0);
            }
            REQUIRE(image[4096 * d.size()] == 0xCC);
            // a range past its allocation, an address of none, a destination too short: refused, in known allocations and in new ones
            memset(image, 0xCC, 4 << 20);
            for (int k : {0, arenas, 119}) {
                auto bad = d;
                bad[k].nbytes = uint64_t(g_allocations[k % arenas].base + size - static_cast<uint8_t *>(bad[k].dev_ptr)) + 1;
                REQUIRE(pack(bad.data(), bad.size(), image, 4 << 20, nullptr) == CKPT_EINVAL);
                bad = d;
                bad[k].dev_ptr = &bad;
                REQUIRE(pack(bad.data(), bad.size(), image, 4 << 20, nullptr) == CKPT_EINVAL);
            }
            REQUIRE(pack(d.data(), d.size(), image + (4 << 20) - 8192, 120 * 4096, nullptr) == CKPT_EINVAL);
            for (uint64_t i = 0; i < 4 << 20; i++) REQUIRE(image[i] == 0xCC);
        }
    for (auto &a : g_allocations) free(a.base);
    printf("ok pack image\n");
    return 0;
}
