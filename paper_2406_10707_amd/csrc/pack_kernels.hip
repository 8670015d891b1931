// Pack and scatter kernels for gfx950: pure byte movement between scattered tensors and the
// contiguous, 4 KiB-aligned staging image of the checkpoint's data region. HBM-bound.
//
// One wavefront (64 lanes) walks one tile of the descriptor table: up to 32 KiB of destination,
// 16 bytes per lane per step, 1 KiB per wavefront step. The staging side is always 16-byte aligned. The
// tensor side is aligned to its element size only. The pack kernel reads it with 16-byte vector loads at the
// tensor's own addresses (the target supports unaligned vector loads), each of which lies wholly inside the
// tensor; the one word that holds the tensor's last bytes is built from aligned 16-byte words and byte shifts
// (v_alignbyte). The scatter kernel writes it the same way, its last bytes one by one: nothing outside a tensor is
// ever read past its 16-byte line or written at all.
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>

#include "../../include/ckpt.h"
#include "kernel_util.hpp"
#include "tile_batch.hpp"

namespace dsllm {

// tuning constants (overridable at compile time for sweeps)
#ifndef DSLLM_PACK_WAVES_PER_BLOCK
#define DSLLM_PACK_WAVES_PER_BLOCK 4
#endif
// Wave priority of the pack waves (s_setprio, 0..3). The kernel runs beside the training
// step's GEMM waves on the same compute units; with the highest issue priority a pack launch takes
// 4.5 % less time under a running GEMM loop (measured: 5.44 -> 5.68 TB/s per launch) and the step as a
// whole loses less, because the short burst of memory traffic is over sooner.
#ifndef DSLLM_PACK_PRIO
#define DSLLM_PACK_PRIO 3
#endif
// Ten loads in flight need 54 vector registers, which are handed out as 56 (eight need 46, eleven 58 = 64).
#ifndef DSLLM_PACK_ROLL
#define DSLLM_PACK_ROLL 10
#endif
constexpr uint64_t kPackTileBytes = 32 * 1024;   // the planner's tile size (plan.hpp: kTileBytes)
constexpr int kWavesPerBlock = DSLLM_PACK_WAVES_PER_BLOCK;
constexpr int kBlock = 64 * kWavesPerBlock;
constexpr int kRoll = DSLLM_PACK_ROLL;                 // pack: 16-byte words per lane in flight

// bytes [sh, sh+16) of the 32-byte string lo||hi, for sh = 4*W + b, 1 <= sh <= 15
template <int W>
__device__ __forceinline__ u32x4 funnel(u32x4 lo, u32x4 hi, uint32_t b) {
    uint32_t w[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
    u32x4 o;
    o.x = __builtin_amdgcn_alignbyte(w[W + 1], w[W + 0], b);
    o.y = __builtin_amdgcn_alignbyte(w[W + 2], w[W + 1], b);
    o.z = __builtin_amdgcn_alignbyte(w[W + 3], w[W + 2], b);
    o.w = __builtin_amdgcn_alignbyte(w[W + 4], w[W + 3], b);
    return o;
}

// keep the first `keep` bytes (0..16) of v, zero the rest
__device__ __forceinline__ u32x4 keep_bytes(u32x4 v, uint32_t keep) {
    uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int j = 0; j < 4; j++) {
        uint32_t lo = 4u * j;
        if (keep <= lo) w[j] = 0;
        else if (keep < lo + 4) w[j] &= (1u << (8 * (keep - lo))) - 1u;
    }
    return u32x4{w[0], w[1], w[2], w[3]};
}

// ---------------------------------------------------------------- pack: tensors -> staging

// The 16-byte word that holds a tensor's last bytes: `tail` (1..15) bytes from `addr` on, then zeros. It never comes from
// an unaligned load (that would read up to 15 bytes past the tensor, possibly into an unmapped page): it is put
// together from the one or two aligned words that hold those bytes.
__device__ __forceinline__ u32x4 tail_word(uint64_t addr, uint32_t tail) {
    const uint32_t sh = uint32_t(addr) & 15, b = sh & 3;
    const u32x4 *s = reinterpret_cast<const u32x4 *>(addr - sh);
    u32x4 v = ld16(s);
    if (sh != 0) {
        const u32x4 w1 = (sh + tail > 16) ? ld16(s + 1) : u32x4{0, 0, 0, 0};
        switch (sh >> 2) {
            case 0: v = funnel<0>(v, w1, b); break;
            case 1: v = funnel<1>(v, w1, b); break;
            case 2: v = funnel<2>(v, w1, b); break;
            default: v = funnel<3>(v, w1, b); break;
        }
    }
    return keep_bytes(v, tail);
}

// Output word j (16 bytes at du + 16 j) = the 16 bytes at su + 16 j: one group of 64 U words starting at word g, every
// load of the group issued before its first store. su may have any alignment: the target supports unaligned vector
// loads (a 16-byte load at a 2-byte-aligned address is a single global_load_dwordx4), and all 16 bytes of every
// word lie inside the tensor, so nothing outside it is read. The same holds for the stores.
template <int U>
__device__ __forceinline__ void copy_group(const uint8_t *su, uint8_t *du, uint32_t g, uint32_t lane) {
    // one 64-bit base per side and constant offsets: a 32-bit word index per load would cost an address register pair each
    const uint8_t *sl = su + 16ull * (g + lane);
    uint8_t *dl = du + 16ull * (g + lane);
    u32x4 v[U];
#pragma unroll
    for (int u = 0; u < U; u++) v[u] = ld16_unaligned(sl + 1024 * u);
#pragma unroll
    for (int u = 0; u < U; u++) st16_unaligned(dl + 1024 * u, v[u]);
}

// The n words of a tile at su to du (same contract as copy_group; du may have any alignment too). A full tile (2048 words, 32
// per lane) runs as a rolling pipeline: kRoll loads are issued, then every store is followed at once by the load
// that reuses its registers, so kRoll loads stay in flight from the first word of the tile to the last instead
// of draining after every group. The fences keep the compiler from hoisting all loads to the front, which costs
// a hundred registers more. Shorter tiles (the last tile of a tensor, small tensors) go group by group.
//
// Measured on MI355X against a shape that keeps the whole tile (32 loads per lane, 138 registers) in flight:
// alone on the card the two are within 1 % of each other (0.75 of the HBM peak on aligned tensors, 0.71 on the
// fragmented workload); beside a matrix kernel that leaves 64 registers per lane free only this one finds room on the
// SIMDs (0.71 to 0.74 against 0.45 to 0.55). Against a kernel that writes one KiB per wave in address order, as
// pack_batch_kernel does, it is slower alone (6.02 against 6.66 TB/s aligned, 5.68 against 6.18 fragmented), equal beside a
// 1300 TFLOP/s GEMM loop on aligned tensors (5.87) and faster there on fragmented ones (5.70 against 4.9): the
// engine's launches run beside the training step, so they use this one.
__device__ __forceinline__ void copy_rolling(const uint8_t *su, uint8_t *du, uint32_t n, uint32_t lane) {
    uint32_t g = 0;
#pragma unroll 1
    for (; g + 2048 <= n; g += 2048) {
        const uint8_t *sl = su + 16ull * (g + lane);
        uint8_t *dl = du + 16ull * (g + lane);
        u32x4 v[kRoll];
#pragma unroll
        for (int u = 0; u < kRoll; u++) v[u] = ld16_unaligned(sl + 1024 * u);
#if defined(__HIP_DEVICE_COMPILE__)
        __builtin_amdgcn_sched_barrier(0);
#endif
#pragma unroll
        for (int k = 0; k < 32; k++) {
            st16_unaligned(dl + 1024 * k, v[k % kRoll]);
            if (k + kRoll < 32) v[k % kRoll] = ld16_unaligned(sl + 1024 * (k + kRoll));
#if defined(__HIP_DEVICE_COMPILE__)
            __builtin_amdgcn_sched_barrier(0);
#endif
        }
    }
#pragma unroll 1
    for (; g + 64 * 8 <= n; g += 64 * 8) copy_group<8>(su, du, g, lane);
    if (g + 64 * 4 <= n) { copy_group<4>(su, du, g, lane); g += 64 * 4; }
    if (g + 64 * 2 <= n) { copy_group<2>(su, du, g, lane); g += 64 * 2; }
    if (g + 64 <= n) { copy_group<1>(su, du, g, lane); g += 64; }
    const uint32_t i = g + lane;
    if (i < n) st16_unaligned(du + 16ull * i, ld16_unaligned(su + 16ull * i));
}

// Output words [lo, hi) of one tile (16-byte words of its destination): source bytes where the tile has them,
// the masked tail word, zero padding behind it. All lanes of the wave in step; the tile's fields are wave-uniform.
__device__ __forceinline__ void pack_range(uint64_t src, u32x4 *dst, uint32_t copy_bytes, uint32_t total_bytes, uint32_t lo, uint32_t hi,
                                           uint32_t lane) {
    const uint32_t n_total = total_bytes >> 4;   // 16-byte words to write
    const uint32_t n_full = copy_bytes >> 4;     // of which fully covered by source bytes
    const uint32_t tail = copy_bytes & 15;       // source bytes in word n_full
    if (hi > n_total) hi = n_total;
    if (lo >= hi) return;
    const uint32_t c_hi = hi < n_full ? hi : n_full;            // copy words [lo, c_hi)
    const uint32_t n = c_hi > lo ? c_hi - lo : 0;
    const bool own_tail = tail && lo <= n_full && n_full < hi;  // the range that holds word n_full writes the tail

    // the n words that lie wholly inside the tensor, read at the tensor's own (possibly misaligned) addresses
    copy_rolling(reinterpret_cast<const uint8_t *>(src) + 16ull * lo, reinterpret_cast<uint8_t *>(dst + lo), n, lane);
    if (own_tail && lane == 0) st16(dst + n_full, tail_word(src + 16ull * n_full, tail));
    // zero padding after the tensor's last byte
    const uint32_t z0 = n_full + (tail ? 1u : 0u);
    for (uint32_t i = (z0 > lo ? z0 : lo) + lane; i < hi; i += 64) st16(dst + i, u32x4{0, 0, 0, 0});
}

__global__ __launch_bounds__(kBlock) void pack_kernel(const ckpt_tile *__restrict__ tiles, uint64_t n_tiles,
                                                     uint8_t *__restrict__ slot_base, uint64_t slot_data_off) {
    const uint32_t lane = threadIdx.x & 63;
#if defined(__HIP_DEVICE_COMPILE__) && DSLLM_PACK_PRIO > 0
    __builtin_amdgcn_s_setprio(DSLLM_PACK_PRIO);
#endif
    // The wavefront's number within the block is made uniform first: the descriptor address is then a
    // scalar value and the descriptor arrives through scalar loads (read-only path, no vector-memory
    // round trip before the first data load); measured, this closes the gap to a table-free copy.
    const uint64_t t = uint64_t(blockIdx.x) * kWavesPerBlock + uniform_u32(threadIdx.x >> 6);
    if (t >= n_tiles) return;
    const ckpt_tile *tp = tiles + t;
    const uint64_t src = uniform_u64(tp->src);
    const uint64_t dst_off = uniform_u64(tp->dst_off);
    u32x4 *dst = reinterpret_cast<u32x4 *>(slot_base + (dst_off - slot_data_off));
    pack_range(src, dst, uniform_u32(tp->copy_bytes), uniform_u32(tp->total_bytes), 0, uint32_t(kPackTileBytes / 16), lane);
}

// The image of a batch of pieces of tensors without a tile table: the pieces travel in the kernel arguments. The
// image is a sequence of 4 KiB pages, each of one piece only; a block of ONE wave writes one KiB of one page, 16 bytes
// per lane, and finds its piece through scalar loads of the arguments (the same cache lines for every wave of a compute unit).
//
// HBM-bound. What limits a copy here is the order in which requests reach the memory: with one load and one store per
// lane and blocks that are handed out in address order, the whole chip sweeps source and image in one narrow front.
// Measured on MI355X, read + write: 6.76 TB/s on 11 GB of large aligned tensors, 6.7 on 1.7 GB in 592 tensors, 6.3 on
// 3.7 GB of misaligned fragments, where a wave that walks 32 KiB on its own (pack_kernel, and a kernel that writes its
// table before it) reaches 5.73, 5.47 and 5.13. More words per lane widen the front and lose (2: 5.3 to 6.1; 4: 5.9 to
// 6.1), four waves per block lose 5 % on aligned tensors (6.43) and win 1 % on fragments. On small lists the table was
// the cost: 112 tensors of 0.4 MB took three kernels, 28 us back to back.
//
// RUNS: of every 64 KiB, each XCD takes eight in a row instead of every eighth (consecutive blocks go to the eight XCDs in
// turn). Of a tensor that does not start on a 128-byte line every wave's KiB ends in the middle of one, which the next wave
// reads again; on the same XCD it finds it in that XCD's L2. Measured on MI355X: 3.7 GB of misaligned fragments 1399 -> 1362 us, 0.6
// GB of smaller ones 574 -> 553 (runs of 4: 1384, 562; of 16: 1390, 553). Aligned tensors share no lines and lose by the
// wider front: 1321 -> 1339 us, 11 GB of large ones 3368 -> 3525.
template <bool RUNS, int N>
__global__ __launch_bounds__(64) void pack_batch_kernel(PackArgs<N> args, uint8_t *__restrict__ image) {
    const uint32_t turn = blockIdx.x % 64, kib = RUNS ? blockIdx.x - turn + turn % 8 * 8 + turn / 8 : blockIdx.x;
    const uint32_t page = kib / 4, at = (kib % 4) * 1024 + 16 * threadIdx.x;
    if (page >= args.pages) return;
    const PackSource s = args.of(page);
    u32x4 v = {0, 0, 0, 0};                                    // padding behind the tensor's last byte
    if (at + 16 <= s.bytes) v = ld16_unaligned(reinterpret_cast<const uint8_t *>(s.src + at));
    else if (at < s.bytes) v = tail_word(s.src + at, s.bytes - at);
    st16(reinterpret_cast<u32x4 *>(image + kPackPage * page + at), v);
}

// ---------------------------------------------------------------- scatter: staging -> tensors

// The pack kernel's way back: the same pipeline with the tensor's own addresses on the side of the stores. HBM-bound, at 5 TB/s read +
// write in launches of 64 MiB (2048 waves). Funnels that put together words aligned at the destination, the form before, read
// every staging word twice: us per launch of 64 MiB, before and now, misaligned fragments 34.8 -> 28.9, 1.7 GB in 592 misaligned
// tensors 31.5 -> 27.4, aligned 27.2 -> 26.5; 12,000 tensors of 40 to 12,000 bytes 17.6 -> 14.9.
__global__ __launch_bounds__(kBlock) void scatter_kernel(const ckpt_tile *__restrict__ tiles, uint64_t n_tiles,
                                                        const uint8_t *__restrict__ slot_base, uint64_t slot_data_off) {
    const uint32_t lane = threadIdx.x & 63;
    const uint64_t t = uint64_t(blockIdx.x) * kWavesPerBlock + uniform_u32(threadIdx.x >> 6);   // uniform: scalar descriptor loads
    if (t >= n_tiles) return;
    const ckpt_tile *tp = tiles + t;
    const uint64_t dstp = uniform_u64(tp->src);
    const uint64_t off = uniform_u64(tp->dst_off);
    const uint32_t nbytes = uniform_u32(tp->copy_bytes);
    if (nbytes == 0) return;
    const uint8_t *src = slot_base + (off - slot_data_off);   // 16-byte aligned
    uint8_t *dst = reinterpret_cast<uint8_t *>(dstp);
    const uint32_t n_full = nbytes >> 4;
    copy_rolling(src, dst, n_full, lane);
    // bytes behind the last full word: the rest of that word belongs to another tensor and may be written concurrently
    const uint32_t tail = nbytes & 15;
    if (lane < tail) dst[16ull * n_full + lane] = src[16ull * n_full + lane];
}

// ---------------------------------------------------------------- launchers (host)

// A launch of fewer pages takes little more than a launch, whatever the order (see pack_batch_kernel).
#ifndef DSLLM_PACK_RUNS_FROM
#define DSLLM_PACK_RUNS_FROM 2048
#endif

// Groups of pages are made from 4 MiB on: 592 tensors of 50 MB 23.8 -> 20.9 us, 288 of 250 MB 94.9 -> 92.3, 2400 of 4.3 GB (misaligned)
// 1384 -> 1368; with fewer pages the host takes longer than the kernel (316 tensors of 3.7 MB 4.7 us either way). Not where more than half of the pages
// are in large pieces, on which waves that know their piece sooner gain little and make the front of addresses wider (as far as one can
// tell from outside; in the Adam kernel more waves than the memory needs do the same). In order the line is at 64 MiB, without -> with groups,
// over two cards: pieces of 4 MiB 1533 -> 1475, 17 MiB 2123 -> 2084 and 2102 -> 2097, 40 MiB 3098 -> 3056 and 3078 -> 3067, 75 MiB
// 3344 -> 3309, 144 of 32 to 172 MiB 3345 -> 3314 and 3317 -> 3327, 1 GiB 3158 -> 3170 and 3138 -> 3181; bisection of more than 320 pieces always takes longer
// (one of 4 GB with 1200 of 64 KiB 1324 -> 1313). In runs at 8 MiB: 1 MiB 416 -> 407,
// 2 MiB 811 -> 799, 6 MiB 1993 -> 1985, 10 MiB even, 17 MiB 2240 -> 2255, 40 MiB 3279 -> 3297; one piece of 8 GB with 1000 of a MiB 3002 -> 3043, of
// 4 GB with 1200 of 64 KiB 1370 -> 1391.
#ifndef DSLLM_PACK_GROUPS_FROM
#define DSLLM_PACK_GROUPS_FROM 1024
#endif
constexpr uint32_t kLargePiece = 16384, kLargePieceRuns = 2048;      // pages: what a launch in order, or in runs, calls a large piece

// Writes the pieces of `bt` to `image`, which begins with the page of the batch's first piece. A batch without pieces
// launches one block of every kernel that finds nothing to do (it makes the runtime load the kernels' code). The arguments
// have four sizes, as a launch takes the host longer with more bytes of them: 12 tensors 3.4 us with 4 KB, 3.1 with 0.5.
template <int MOST>
static hipError_t launch_batch(PackBatchOf<MOST> &bt, void *image, hipStream_t stream) {
    const uint32_t pages = bt.pages;
    uint32_t off_lines = 0;                      // pages of pieces that do not start on a 128-byte line
    uint32_t in_large = 0, in_large_runs = 0;    // of large pieces
    if (pages >= DSLLM_PACK_RUNS_FROM)
        for (uint32_t k = 0; k < bt.count; k++) {
            const uint32_t n = bt.first_page[k + 1] - bt.first_page[k];
            if (bt.src(k) % 128) off_lines += n;
            if (n <= kLargePieceRuns) continue;
            in_large_runs += n;
            if (n > kLargePiece) in_large += n;
        }
    const bool runs = off_lines > pages / 2 || !pages, in_order = off_lines <= pages / 2;
    const bool large = in_order ? in_large > pages / 2 && bt.count <= uint32_t(kPackBatch) : in_large_runs > pages / 2;
    bt.make_groups(pages >= DSLLM_PACK_GROUPS_FROM && !large);
    auto launch = [&](const auto &args, auto runs_kernel, auto kernel) {
        const unsigned kib = pages ? pages * 4 : 1;
        if (runs) hipLaunchKernelGGL(runs_kernel, dim3((kib + 63) / 64 * 64), dim3(64), 0, stream, args, static_cast<uint8_t *>(image));
        if (in_order) hipLaunchKernelGGL(kernel, dim3(kib), dim3(64), 0, stream, args, static_cast<uint8_t *>(image));
    };
    if (bt.count <= 32) launch(bt.template shorter<32>(), pack_batch_kernel<true, 32>, pack_batch_kernel<false, 32>);
    if ((bt.count > 32 && bt.count <= 128) || !pages) launch(bt.template shorter<128>(), pack_batch_kernel<true, 128>, pack_batch_kernel<false, 128>);
    if ((bt.count > 128 && bt.count <= uint32_t(kPackBatch)) || !pages)
        launch(bt.template shorter<kPackBatch>(), pack_batch_kernel<true, kPackBatch>, pack_batch_kernel<false, kPackBatch>);
    if constexpr (MOST > kPackBatch)
        if (bt.count > uint32_t(kPackBatch) || !pages) launch(static_cast<const PackArgs<MOST> &>(bt), pack_batch_kernel<true, MOST>, pack_batch_kernel<false, MOST>);
    return hipGetLastError();
}
hipError_t launch_pack_batch(PackBatch &bt, void *image, hipStream_t stream) { return launch_batch(bt, image, stream); }
hipError_t launch_pack_batch(LongPackBatch &bt, void *image, hipStream_t stream) { return launch_batch(bt, image, stream); }

static inline unsigned grid_for(uint64_t n_tiles) { return unsigned((n_tiles + kWavesPerBlock - 1) / kWavesPerBlock); }

hipError_t launch_pack(const ckpt_tile *dev_tiles, uint64_t n_tiles, void *slot_base, uint64_t slot_data_off, hipStream_t stream,
                       hipEvent_t t_start, hipEvent_t t_stop) {
    if (n_tiles == 0) return hipSuccess;
    if (t_start || t_stop)   // the events take the kernel's own start and end, not the moments two host calls around it were processed
        hipExtLaunchKernelGGL(pack_kernel, dim3(grid_for(n_tiles)), dim3(kBlock), 0, stream, t_start, t_stop, 0, dev_tiles, n_tiles,
                              static_cast<uint8_t *>(slot_base), slot_data_off);
    else
        hipLaunchKernelGGL(pack_kernel, dim3(grid_for(n_tiles)), dim3(kBlock), 0, stream, dev_tiles, n_tiles, static_cast<uint8_t *>(slot_base),
                           slot_data_off);
    return hipGetLastError();
}

hipError_t launch_scatter(const ckpt_tile *dev_tiles, uint64_t n_tiles, const void *slot_base, uint64_t slot_data_off, hipStream_t stream) {
    if (n_tiles == 0) return hipSuccess;
    hipLaunchKernelGGL(scatter_kernel, dim3(grid_for(n_tiles)), dim3(kBlock), 0, stream, dev_tiles, n_tiles,
                       static_cast<const uint8_t *>(slot_base), slot_data_off);
    return hipGetLastError();
}

}  // namespace dsllm
