// Kernels of the data reduction (format version 2): a bf16 working copy that is the round-to-nearest-even
// of its f32 master weights is not stored. verify_pairs_kernel checks, on the captured state, that every
// declared pair really is one (so that leaving the copy out loses nothing); derive_pairs_kernel recomputes
// the copies after a restore. Both are HBM-bound streaming kernels: 6 bytes per element read (verify),
// 4 read + 2 written (derive). The rounding is integer arithmetic on the bit pattern, the same definition
// the file format states, so both sides of a comparison take the decision in the same (exact) arithmetic.
//
// A block of four waves takes 4096 elements of a tile, each lane four groups of four: one 16-byte access to the f32 side and
// one 8-byte access to the bf16 side each, all loads before the first use. The accesses are made at the tensors' own
// addresses (aligned to their element size only; the target allows unaligned vector accesses, and every one lies inside
// its tensor). Measured: 202 M aligned elements, verify 186 -> 182 us (6.7 TB/s), derive 219 -> 198; 68 M elements of
// flattened buffers, where element-wise accesses were the general case, 99 -> 62 and 109 -> 72. Fewer groups per lane
// (one: 174 and 177 us aligned) leave three blocks in four without work on tensors of a thousand elements (14 -> 22 us;
// this shape 10.6).
#include "kernel_util.hpp"
#include "plan.hpp"

namespace dsllm {

constexpr uint32_t kPairBlock = 256, kPairUnroll = 4;
constexpr uint32_t kPairBlockElems = 4 * kPairBlock * kPairUnroll;
constexpr uint32_t kPairBlocksPerTile = kPairTileElems / kPairBlockElems;
static_assert(kPairBlocksPerTile * kPairBlockElems == kPairTileElems, "blocks divide a tile");

__device__ __forceinline__ uint32_t bf16_rne(uint32_t u) {
    const uint32_t nan = (u >> 16) | 0x0040u;
    const uint32_t rounded = (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
    return ((u & 0x7FFFFFFFu) > 0x7F800000u ? nan : rounded) & 0xFFFFu;
}

// the four bf16 patterns of four f32 patterns, packed as they lie in memory
__device__ __forceinline__ u32x2 bf16_rne4(u32x4 m) {
    return u32x2{bf16_rne(m.x) | (bf16_rne(m.y) << 16), bf16_rne(m.z) | (bf16_rne(m.w) << 16)};
}

// 8 bytes at any byte address; all of them must lie inside the tensor
typedef u32x2 u32x2_bytealigned __attribute__((aligned(1)));
__device__ __forceinline__ u32x2 ld8_unaligned(const uint8_t *p) { return __builtin_nontemporal_load((const u32x2_bytealigned DSLLM_GLOBAL *)p); }
__device__ __forceinline__ void st8_unaligned(uint8_t *p, u32x2 v) { __builtin_nontemporal_store(v, (u32x2_bytealigned DSLLM_GLOBAL *)p); }

// WRITE = false: *mismatch is set to 1 if any element of a bf16 tensor differs from the rounding of its source.
// WRITE = true: the bf16 tensors are overwritten with the rounding of their sources.
template <bool WRITE>
__device__ __forceinline__ void pairs_body(const PairTile *__restrict__ tiles, uint32_t *mismatch) {
    const PairTile *tp = tiles + blockIdx.x / kPairBlocksPerTile;      // uniform: scalar descriptor loads
    const uint8_t *f32 = reinterpret_cast<const uint8_t *>(uniform_u64(tp->f32_addr));
    uint8_t *bf16 = reinterpret_cast<uint8_t *>(uniform_u64(tp->bf16_addr));
    const uint32_t count = uniform_u32(tp->count);
    const uint32_t first = (blockIdx.x % kPairBlocksPerTile) * kPairBlockElems + 4 * threadIdx.x;
    u32x4 v[kPairUnroll];
    u32x2 have[kPairUnroll];
    bool bad = false;
#pragma unroll
    for (uint32_t u = 0; u < kPairUnroll; u++) {
        const uint32_t e = first + 4 * kPairBlock * u;
        if (e + 4 > count) continue;
        v[u] = ld16_unaligned(f32 + 4ull * e);
        if (!WRITE) have[u] = ld8_unaligned(bf16 + 2ull * e);
    }
#pragma unroll
    for (uint32_t u = 0; u < kPairUnroll; u++) {
        uint32_t e = first + 4 * kPairBlock * u;
        if (e + 4 <= count) {
            const u32x2 want = bf16_rne4(v[u]);
            if (WRITE) st8_unaligned(bf16 + 2ull * e, want);
            else bad |= (want.x != have[u].x) | (want.y != have[u].y);
        } else {
            for (; e < count; e++) {      // up to three elements behind the last group of four
                const uint32_t want = bf16_rne(reinterpret_cast<const uint32_t *>(f32)[e]);
                uint16_t *p = reinterpret_cast<uint16_t *>(bf16) + e;
                if (WRITE) *p = uint16_t(want);
                else bad |= want != *p;
            }
        }
    }
    if (!WRITE && bad) *mismatch = 1;     // every lane that found a difference stores the same value: no atomics needed
}

__global__ __launch_bounds__(kPairBlock) void verify_pairs_kernel(const PairTile *__restrict__ tiles, uint32_t *mismatch) { pairs_body<false>(tiles, mismatch); }

__global__ __launch_bounds__(kPairBlock) void derive_pairs_kernel(const PairTile *__restrict__ tiles) { pairs_body<true>(tiles, nullptr); }

__global__ void clear_word_kernel(uint32_t *word) { *word = 0; }

// a grid has fewer than 2^32 work-items: tables longer than this go in several launches
constexpr uint64_t kPairTilesPerLaunch = 1u << 22;

// Clears the flag and checks every pair; the flag is 1 afterwards if any pair does not hold.
hipError_t launch_verify_pairs(const PairTile *dev_tiles, uint64_t n_tiles, uint32_t *dev_flag, hipStream_t stream) {
    hipLaunchKernelGGL(clear_word_kernel, dim3(1), dim3(1), 0, stream, dev_flag);
    for (uint64_t t = 0; t < n_tiles; t += kPairTilesPerLaunch) {
        const uint64_t n = n_tiles - t < kPairTilesPerLaunch ? n_tiles - t : kPairTilesPerLaunch;
        hipLaunchKernelGGL(verify_pairs_kernel, dim3(unsigned(n * kPairBlocksPerTile)), dim3(kPairBlock), 0, stream, dev_tiles + t, dev_flag);
    }
    return hipGetLastError();
}

hipError_t launch_derive_pairs(const PairTile *dev_tiles, uint64_t n_tiles, hipStream_t stream) {
    for (uint64_t t = 0; t < n_tiles; t += kPairTilesPerLaunch) {
        const uint64_t n = n_tiles - t < kPairTilesPerLaunch ? n_tiles - t : kPairTilesPerLaunch;
        hipLaunchKernelGGL(derive_pairs_kernel, dim3(unsigned(n * kPairBlocksPerTile)), dim3(kPairBlock), 0, stream, dev_tiles + t);
    }
    return hipGetLastError();
}

}  // namespace dsllm
