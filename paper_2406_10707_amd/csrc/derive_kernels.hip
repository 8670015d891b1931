// Kernels of the data reduction (format version 2): a bf16 working copy that is the round-to-nearest-even
// of its f32 master weights is not stored. verify_pairs_kernel checks, on the captured state, that every
// declared pair really is one (so that leaving the copy out loses nothing); derive_pairs_kernel recomputes
// the copies after a restore. Both are HBM-bound streaming kernels: 6 bytes per element read (verify),
// 4 read + 2 written (derive). The rounding is integer arithmetic on the bit pattern, the same definition
// the file format states, so both sides of a comparison take the decision in the same (exact) arithmetic.
//
// A block takes a work item of up to 4096 elements, four waves with four groups of four elements per lane (check) or eight waves with
// two (regeneration): per group one 16-byte access to the f32 side and one 8-byte access to the bf16 side, all loads before the first
// use and none of them under a mask (a lane behind the last whole group takes the item's last four elements instead). Work
// items of up to 512 elements go one to a wave. The accesses are made at the tensors' own addresses (aligned to their element
// size only; the target allows unaligned vector accesses, and every one lies inside its tensor).
//
// Where many tensors are short, blocks are what costs, hence a wave each for those. Measured in us, check and regeneration, with
// one wave per 8192 elements (element-wise accesses where a tensor is not aligned) / two blocks of four waves per 8192
// elements, masked / now:
//   202 M aligned elements               184, 219 / 178, 200 / 177, 187 (6.9 and 6.5 TB/s)
//   68 M elements of flattened buffers   107, 109 / 61, 73 / 62, 69
//   4000 tensors of about 4100           42, 32 / 24, 27 / 18, 20.5
//   4000 of about 1000                   16, 12 / 12, 12.4 / 7.6, 9.5
//   the same, aligned                    8.4, 8.7 / 11.4, 11.9 / 7.4, 9.2
//   20,000 of about 100                  8.3, 8.0 / 31, 24 / 6.6, 7.9
// The check runs beside the training step. There blocks of eight waves find room later: 1.0 G aligned elements beside a GEMM
// loop 1014 us, 1102 to 1195 with eight waves, 1009 masked, 1054 with a wave per 8192. The regeneration runs on an idle card,
// where eight waves are 3 to 5 % faster than four. The bound between a block and a wave (measured with four waves): 2000
// tensors of 1000 to 4000 take 8.8 and 10.1 with 512 elements, 9.9 and 10.6 with 1024, 9.6 and 10.3 with 256.
#include "kernel_util.hpp"
#include "plan.hpp"

namespace dsllm {

constexpr uint32_t kVerifyWaves = 4, kDeriveWaves = 8;     // per block
static_assert(kPairSmallElems == 4 * 2 * 64, "a wave's lanes take two groups of four");

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

// WRITE = false: returns whether an element of the bf16 tensor differs from the rounding of its source.
// WRITE = true: the bf16 tensor is overwritten with the rounding of its source.
// Of the work item's groups of four elements this lane takes GROUPS: number `lane`, `lane` + `lanes`, ... SKIP: groups that no lane
// of the `lanes` has are passed over by a uniform branch (worth it only where items are often short).
template <bool WRITE, uint32_t GROUPS, bool SKIP>
__device__ __forceinline__ bool pair_share(const PairTile *tp, uint32_t lane, uint32_t lanes) {
    const uint8_t *f32 = reinterpret_cast<const uint8_t *>(uniform_u64(tp->f32_addr));   // uniform: scalar descriptor loads
    uint8_t *bf16 = reinterpret_cast<uint8_t *>(uniform_u64(tp->bf16_addr));
    const uint32_t count = uniform_u32(tp->count);
    bool bad = false;
    if (count < 4) {
        if (lane < count) {
            const uint32_t want = bf16_rne(reinterpret_cast<const uint32_t *>(f32)[lane]);
            uint16_t *p = reinterpret_cast<uint16_t *>(bf16) + lane;
            if (WRITE) *p = uint16_t(want);
            else bad = want != *p;
        }
        return bad;
    }
    // A lane whose group does not end inside the item takes the last four elements: those of the ragged end are among them,
    // the others are some lane's already (compared twice, or written twice with the same bits).
    auto place = [&](uint32_t e) { return e + 4 <= count ? e : count - 4; };
    u32x4 v[GROUPS];
    u32x2 have[GROUPS];
#pragma unroll
    for (uint32_t u = 0; u < GROUPS; u++) {
        if (SKIP && 4 * lanes * u >= count) continue;
        const uint32_t e = place(4 * (lane + lanes * u));
        v[u] = ld16_unaligned(f32 + 4ull * e);
        if (!WRITE) have[u] = ld8_unaligned(bf16 + 2ull * e);
    }
#pragma unroll
    for (uint32_t u = 0; u < GROUPS; u++) {
        if (SKIP && 4 * lanes * u >= count) continue;
        const uint32_t group = 4 * (lane + lanes * u);
        const u32x2 want = bf16_rne4(v[u]);
        if (!WRITE) bad |= (want.x != have[u].x) | (want.y != have[u].y);
        else if (group < count) st8_unaligned(bf16 + 2ull * place(group), want);
    }
    return bad;
}

// Block b of a launch: work item b while those are not small, WAVES small ones after that.
template <bool WRITE, uint32_t WAVES>
__device__ __forceinline__ bool pair_block(const PairTile *__restrict__ tiles, uint32_t n_blocks, uint32_t n_tiles) {
    constexpr uint32_t GROUPS = kPairTileElems / (4 * 64 * WAVES);
    static_assert(GROUPS * 4 * 64 * WAVES == kPairTileElems && GROUPS >= 2, "a block's lanes take whole groups");
    if (blockIdx.x < n_blocks) {
        const PairTile *tp = tiles + blockIdx.x;
        if (GROUPS > 2 && uniform_u32(tp->count) > 4 * 2 * 64 * WAVES) return pair_share<WRITE, GROUPS, false>(tp, threadIdx.x, 64 * WAVES);
        return pair_share<WRITE, 2, true>(tp, threadIdx.x, 64 * WAVES);
    }
    const uint32_t t = n_blocks + (blockIdx.x - n_blocks) * WAVES + uniform_u32(threadIdx.x >> 6);
    return t < n_tiles && pair_share<WRITE, 2, true>(tiles + t, threadIdx.x & 63, 64);
}

// *mismatch is set to 1 if any element of a bf16 tensor differs from the rounding of its source.
__global__ __launch_bounds__(64 * kVerifyWaves) void verify_pairs_kernel(const PairTile *__restrict__ tiles, uint32_t n_blocks, uint32_t n_tiles, uint32_t *mismatch) {
    if (pair_block<false, kVerifyWaves>(tiles, n_blocks, n_tiles)) *mismatch = 1;   // all that found one store the same value: no atomics needed
}

__global__ __launch_bounds__(64 * kDeriveWaves) void derive_pairs_kernel(const PairTile *__restrict__ tiles, uint32_t n_blocks, uint32_t n_tiles) {
    (void)pair_block<true, kDeriveWaves>(tiles, n_blocks, n_tiles);
}

__global__ void clear_word_kernel(uint32_t *word) { *word = 0; }

// a grid has fewer than 2^32 work-items: longer tables go in several launches
#ifndef DSLLM_PAIR_TILES_PER_LAUNCH
#define DSLLM_PAIR_TILES_PER_LAUNCH (1u << 22)
#endif

// launch(tiles, how many of them are not small, how many there are, blocks)
template <class F>
static void for_pair_launches(const PairTile *tiles, uint64_t n_blocks, uint64_t n_tiles, uint32_t waves, F launch) {
    while (n_tiles) {
        const uint32_t n = uint32_t(n_tiles < DSLLM_PAIR_TILES_PER_LAUNCH ? n_tiles : DSLLM_PAIR_TILES_PER_LAUNCH);
        const uint32_t nb = uint32_t(n_blocks < n ? n_blocks : n);
        launch(tiles, nb, n, nb + (n - nb + waves - 1) / waves);
        tiles += n; n_tiles -= n; n_blocks -= nb;
    }
}

// Clears the flag and checks every pair; the flag is 1 afterwards if any pair does not hold.
hipError_t launch_verify_pairs(const PairTile *dev_tiles, uint64_t n_blocks, uint64_t n_tiles, uint32_t *dev_flag, hipStream_t stream) {
    hipLaunchKernelGGL(clear_word_kernel, dim3(1), dim3(1), 0, stream, dev_flag);
    for_pair_launches(dev_tiles, n_blocks, n_tiles, kVerifyWaves, [&](const PairTile *tiles, uint32_t nb, uint32_t n, unsigned grid) {
        hipLaunchKernelGGL(verify_pairs_kernel, dim3(grid), dim3(64 * kVerifyWaves), 0, stream, tiles, nb, n, dev_flag);
    });
    return hipGetLastError();
}

hipError_t launch_derive_pairs(const PairTile *dev_tiles, uint64_t n_blocks, uint64_t n_tiles, hipStream_t stream) {
    for_pair_launches(dev_tiles, n_blocks, n_tiles, kDeriveWaves, [&](const PairTile *tiles, uint32_t nb, uint32_t n, unsigned grid) {
        hipLaunchKernelGGL(derive_pairs_kernel, dim3(grid), dim3(64 * kDeriveWaves), 0, stream, tiles, nb, n);
    });
    return hipGetLastError();
}

}  // namespace dsllm
