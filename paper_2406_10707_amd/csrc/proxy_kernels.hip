// Synthetic training proxy kernels for gfx950 (see include/ckpt_proxy.h): bf16 MFMA GEMM,
// element-wise Adam step, seeded state fill, flat-buffer word fill/mutate, contiguous copy.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdio.h>
#include <stdint.h>

#include <algorithm>
#include <utility>

#include "../../include/ckpt_proxy.h"
#include "gemm_forms.hpp"

using namespace dsllm;

namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// ------------------------------------------------------------------ counter-based random numbers

__device__ __forceinline__ uint64_t mix(uint64_t x) {
    uint64_t z = x + 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}
__host__ __device__ __forceinline__ uint64_t mix_host(uint64_t x) {
    uint64_t z = x + 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}
static uint64_t stream_key(uint64_t seed, uint64_t tensor, uint64_t tag) { return mix_host(seed ^ mix_host(tensor * 4 + tag)); }

__device__ __forceinline__ float normal_from(uint64_t r) {
    const float u_hi = (float(uint32_t(r >> 40)) + 0.5f) * (1.0f / 16777216.0f);
    const float u_lo = (float(uint32_t(r & 0xFFFFFFu)) + 0.5f) * (1.0f / 16777216.0f);
    return sqrtf(-2.0f * logf(u_hi)) * cosf(6.28318530717958647692f * u_lo);
}

__device__ __forceinline__ uint16_t bf16_rne(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return uint16_t((u >> 16) | 0x0040u);
    return uint16_t((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}

// ------------------------------------------------------------------ state fill and Adam step

__global__ __launch_bounds__(256) void fill_state_kernel(uint16_t *__restrict__ p, float *__restrict__ master, float *__restrict__ m,
                                                        float *__restrict__ v, uint64_t numel, uint64_t k0, uint64_t k1, uint64_t k2) {
    const uint64_t stride = uint64_t(gridDim.x) * blockDim.x;
    for (uint64_t i = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < numel; i += stride) {
        const uint64_t hi = mix(i);
        const float w = 0.02f * normal_from(mix(k0 ^ hi));
        master[i] = w;
        p[i] = bf16_rne(w);
        m[i] = 0.02f * normal_from(mix(k1 ^ hi));
        const float s = 0.001f * normal_from(mix(k2 ^ hi));
        v[i] = s * s;
    }
}

struct AdamArgs { float lr, beta1, beta2, eps, inv_bc1, inv_bc2; };

__device__ __forceinline__ void adam_one(float &w, float &m, float &v, uint64_t key, uint64_t i, const AdamArgs &a) {
    const uint64_t r = mix(key ^ mix(i));
    const float g = 0.001f * (float(uint32_t(r >> 32) >> 8) * (1.0f / 8388608.0f) - 1.0f);     // the generator's 24 upper bits to -1 .. 1
    m = a.beta1 * m + (1.0f - a.beta1) * g;
    v = a.beta2 * v + (1.0f - a.beta2) * (g * g);
    const float mhat = m * a.inv_bc1, vhat = v * a.inv_bc2;
    w = w - a.lr * (mhat / (sqrtf(vhat) + a.eps));
}

// Four elements per lane: 16-byte accesses to master, m, v and 8-byte ones to the bf16 copy, one wave per block, each
// element by one lane of the grid, nothing in a loop. HBM-bound (12 bytes an element read, 14 written). Blocks of one wave handed
// out in address order and non-temporal accesses keep the chip in a narrow front of each of the seven streams: 4096 blocks of four waves striding over
// the tensor with ordinary accesses took 1.06 to 1.13 ms for 202 M elements, this 0.88 with as many waves as there is room for.
// Those are more than the memory needs, and the more there are the wider the front: with twelve to a compute unit
// (kAdamLds, which nothing uses, holds off the others) it takes 0.80 ms = 6.6 TB/s; with 16, 14, 11, 10 and 8: 0.81, 0.80, 0.80, 0.82 and 0.91. (A plain
// copy, with one load a wave, is fastest with all it can have.) The rounding to bf16 is one instruction for two elements, which gives
// the bits of bf16_rne for every f32 pattern, in place of two masked branches an element: 1 M elements 5.9 -> 5.6 us.
__global__ __launch_bounds__(64) void adam_kernel(uint16_t *__restrict__ p, float *__restrict__ master, float *__restrict__ m,
                                                 float *__restrict__ v, uint64_t numel, uint64_t first_quad, uint64_t key, AdamArgs a) {
    const uint64_t n4 = numel >> 2, q = first_quad + uint64_t(blockIdx.x) * 64 + threadIdx.x;
    if (q < n4) {
        const f32x4 w4 = __builtin_nontemporal_load(reinterpret_cast<f32x4 *>(master) + q), m4 = __builtin_nontemporal_load(reinterpret_cast<f32x4 *>(m) + q),
                    v4 = __builtin_nontemporal_load(reinterpret_cast<f32x4 *>(v) + q);
        float w[4] = {w4.x, w4.y, w4.z, w4.w}, mm[4] = {m4.x, m4.y, m4.z, m4.w}, vv[4] = {v4.x, v4.y, v4.z, v4.w};
#pragma unroll
        for (int j = 0; j < 4; j++) adam_one(w[j], mm[j], vv[j], key, 4 * q + j, a);
        const f32x4 w_new{w[0], w[1], w[2], w[3]};
        __builtin_nontemporal_store(w_new, reinterpret_cast<f32x4 *>(master) + q);
        __builtin_nontemporal_store(f32x4{mm[0], mm[1], mm[2], mm[3]}, reinterpret_cast<f32x4 *>(m) + q);
        __builtin_nontemporal_store(f32x4{vv[0], vv[1], vv[2], vv[3]}, reinterpret_cast<f32x4 *>(v) + q);
        __builtin_nontemporal_store(__builtin_bit_cast(u32x2, __builtin_convertvector(w_new, bf16x4)), reinterpret_cast<u32x2 *>(p) + q);
    }
    // ragged tail (numel not a multiple of 4)
    const uint64_t t = (n4 << 2) + q;
    if (t < numel) {
        adam_one(master[t], m[t], v[t], key, t, a);
        p[t] = bf16_rne(master[t]);
    }
}
// Shared memory of a block that has room for twelve beside each other (160 KiB a compute unit, handed out in pieces of 1280 bytes); only for grids
// of an eighth more than the chip's 256 x 32 wave slots, as it costs those that fit them at once, and those a little larger where
// nothing follows: 1 M elements 5.6 -> 6.5 us, one tensor of 2.15 M 14.5 -> 15.8, of 2.25 M 15.8 -> 16.6, of 2.4 M even; twenty of 2.3 M one behind the
// other 12.6 -> 12.0 each, of 2.5 M 13.7 -> 12.9.
constexpr unsigned kAdamLds = 12800, kAdamFreeBlocks = 256 * 36;

// ------------------------------------------------------------------ flat-buffer words, copy

__global__ __launch_bounds__(256) void fill_words_kernel(uint32_t *__restrict__ w, uint64_t n, uint64_t key) {
    const uint64_t stride = uint64_t(gridDim.x) * blockDim.x;
    for (uint64_t i = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += stride) w[i] = uint32_t(mix(key ^ mix(i)));
}

__global__ __launch_bounds__(256) void mutate_words_kernel(uint32_t *__restrict__ w, uint64_t n, uint32_t step) {
    const uint64_t stride = uint64_t(gridDim.x) * blockDim.x;
    for (uint64_t i = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += stride) w[i] = w[i] * 1664525u + 1013904223u + step;
}

// A plain copy, what the pack kernels are compared with: 16 bytes per lane, one wave per block, in address order (6.69 TB/s read +
// write over 8 GiB; waves that each stream 32 KiB pieces with sixteen loads in flight, the form before, 5.87).
__global__ __launch_bounds__(64) void devcopy_kernel(u32x4 *__restrict__ dst, const u32x4 *__restrict__ src, uint64_t n16) {
    const uint64_t i = uint64_t(blockIdx.x) * 64 + threadIdx.x;
    if (i < n16) __builtin_nontemporal_store(__builtin_nontemporal_load(src + i), dst + i);
}

// ------------------------------------------------------------------ bf16 GEMM on the matrix cores

// The kernels below compute C = A * B^T tile by tile with MFMA 16x16x32 (the 32x32x16 form does the same work at a
// higher power: at 8192^3 the card held 1.71 GHz with it at 74 % of the matrix pipe's cycles, and holds 1.73 GHz with
// this one at 84 %). Operand panels go from memory to LDS without passing through registers (buffer loads to LDS, 16
// bytes per lane, counted by vmcnt), 64 K values a step, so that every request is a whole 128-byte line.
//
// LDS layout of a panel: rows of 64 K values, 128 bytes, eight 16-byte pieces; row r keeps piece p at place p ^ f(r), so
// that the rows a fragment read touches lie in different banks (no conflicts measured). The loads write LDS in lane
// order, so the permutation is made on the global side: a lane fetches the piece that belongs at its place.
// A fragments hold 16 consecutive rows, f(r) = bits 1..3 of r. B fragments come in pairs that hold 32 rows as
// 8 (lane / 4) + lane % 4 and that + 4, f(r) = bits 1, 3, 4: with B as the first operand a lane then ends up with eight
// consecutive columns of one row of C, one 16-byte store (8-byte stores of 32-byte pieces cost 3 % of the whole).
#define DSLLM_LDS __attribute__((address_space(3)))
#define DSLLM_GLB __attribute__((address_space(1)))

struct GemmTile { int tm, tn; };

// Which tile a block computes. Consecutive block ids go to different XCDs (8 of them, each with its own L2): each XCD is given
// a contiguous range of tiles, walked in strips 8 tiles tall so that neighbours share A and B panels. With a short K the
// stores of C are what counts, and those go better in block order where 8 does not divide the number of tiles (7808 x 3968 x
// 128 18.2 us, by XCD 18.9).
// The host prepares the divisions: three of them, on scalars, were 90 of the 150 instructions in front of a block's first load
// (and a branch costs some 40 cycles, so there is none). Products of 4 to 6 us take 4 % less than with divisions in the kernel, of
// 6 to 10 us 2 %, of 10 to 20 us 1 % (300 products; 1024 x 3072 x 768 7.7 -> 7.5 us, 896 x 3072 x 64 4.1 -> 3.5); those of
// 3 us are bound by the launches.
struct TileOrder {
    uint32_t xcd_bits, xcd_shift;            // of a block id: its XCD, what is left of it (0, 0: tiles go in the blocks' own order)
    uint32_t each, more;                     // tiles of every XCD; how many XCDs have one tile more
    uint32_t per_strip, strip_inverse;       // tiles of a full strip
    uint32_t full_strips, last_rows, last_inverse;       // the last strip may be less than 8 tall

    static uint32_t inverse(uint32_t d) { return 0xFFFFFFFFu / d; }
    // x / d: the upper half of x times the inverse is that or one less
    static __host__ __device__ __forceinline__ uint32_t divided(uint32_t x, uint32_t d, uint32_t inverse) {
        const uint32_t q = uint32_t((uint64_t(x) * inverse) >> 32);
        return x - q * d >= d ? q + 1 : q;
    }
    TileOrder(uint32_t tiles_m, uint32_t tiles_n, bool by_xcd) {
        const uint32_t n = tiles_m * tiles_n;
        const bool in_order = !by_xcd && n % 8;
        xcd_bits = in_order ? 0 : 7;
        xcd_shift = in_order ? 0 : 3;
        each = n / 8;
        more = n % 8;
        per_strip = 8 * tiles_n;
        strip_inverse = inverse(per_strip);
        full_strips = tiles_m / 8;
        last_rows = tiles_m % 8 ? tiles_m % 8 : 8;
        last_inverse = inverse(last_rows);
    }
};

__device__ __forceinline__ GemmTile gemm_tile(const TileOrder &o) {
    const uint32_t xcd = blockIdx.x & o.xcd_bits, tile = xcd * o.each + min(xcd, o.more) + (blockIdx.x >> o.xcd_shift);
    const uint32_t s = TileOrder::divided(tile, o.per_strip, o.strip_inverse), in_s = tile - s * o.per_strip;
    const uint32_t rows_here = s < o.full_strips ? 8 : o.last_rows;
    const uint32_t col = TileOrder::divided(in_s, rows_here, s < o.full_strips ? 1u << 29 : o.last_inverse);
    return GemmTile{int(8 * s + in_s - col * rows_here), int(col)};
}

// One wave's eight rows of a panel per instruction; NW waves share a panel. KEPT: a lane's offset for each instruction stays in
// a register of its own; otherwise the instruction's part is a scalar addition for every load, which is issued in the shadow
// of a matrix instruction. Where that shadow is short the registers are faster (128 x 128 tiles: 3 %), with 256 x 256 tiles
// slower (2 %). WIDE: 64-bit addresses (the lane's own part made once, the instruction's part uniform), for panels that a
// buffer resource's 32-bit offsets do not span.
template <int BM, int BN, int NW, bool PAIRS, bool KEPT, bool WIDE>
struct PanelLoader {
    static constexpr int LA = BM / 8 / NW, LB = BN / 8 / NW, COUNT = LA + LB;   // instructions per wave and step
    static_assert(LA * 8 * NW == BM && LB * 8 * NW == BN && NW % 4 == 0, "panels divide among the waves, four waves' rows per 32");
    const uint16_t *lane_a, *lane_b;
    __amdgpu_buffer_rsrc_t ra, rb;
    uint32_t row0, piece_a, piece_b, k, wave, lane_off[COUNT];

    __device__ __forceinline__ PanelLoader(const uint16_t *a_panel, const uint16_t *b_panel, int K, int lane, int wave_)
        : row0((lane >> 3) + 8 * wave_), piece_a((lane & 7) ^ ((4 * (wave_ & 1) + (lane >> 4)) & 7)),
          piece_b(PAIRS ? (lane & 7) ^ (((lane >> 4) & 1) | ((wave_ & 3) << 1)) : piece_a), k(uint32_t(K)), wave(wave_) {
        if constexpr (WIDE) {
            lane_a = a_panel + size_t(row0) * k + 8 * piece_a;
            lane_b = b_panel + size_t(row0) * k + 8 * piece_b;
        } else {
            ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(a_panel), 0, uint32_t(BM) * 2u * k, 0x00020000);
            rb = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(b_panel), 0, uint32_t(BN) * 2u * k, 0x00020000);
            if constexpr (KEPT)
#pragma unroll
                for (int i = 0; i < COUNT; i++) lane_off[i] = 2 * ((row0 + 8 * NW * (i < LA ? i : i - LA)) * k + 8 * (i < LA ? piece_a : piece_b));
        }
    }
    // instruction i of step kt into the stage at lds (A panel, then B panel)
    __device__ __forceinline__ void issue(uint16_t *lds, int kt, int i) const {
        const bool of_a = i < LA;
        uint16_t *place = lds + (of_a ? 0 : BM * 64) + (of_a ? i : i - LA) * 512 * NW + 512 * wave;
        const uint32_t piece = of_a ? piece_a : piece_b;
        const int j = of_a ? i : i - LA;
        if constexpr (WIDE) {
            const uint16_t *p = (of_a ? lane_a : lane_b) + (size_t(8 * NW * j) * k + size_t(kt) * 64);
            __builtin_amdgcn_global_load_lds((const DSLLM_GLB void *)p, (DSLLM_LDS void *)place, 16, 0, 0);
        } else if constexpr (KEPT) {
            __builtin_amdgcn_raw_ptr_buffer_load_lds(of_a ? ra : rb, (DSLLM_LDS void *)place, 16, lane_off[i], 128 * kt, 0, 0);
        } else {
            __builtin_amdgcn_raw_ptr_buffer_load_lds(of_a ? ra : rb, (DSLLM_LDS void *)place, 16, 2 * (row0 * k + 8 * piece), 16 * NW * j * k + 128 * kt, 0, 0);
        }
    }
};

// This wave's loads are in LDS but for the latest N, its LDS reads are over, and every wave of the block is here.
template <int N>
__device__ __forceinline__ void wait_loads_and_meet() {
    static_assert(N >= 0 && N < 64, "vmcnt has six bits");
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

__device__ __forceinline__ void store_columns(uint16_t *c, f32x4 lo, f32x4 hi) {
    const bf16x4 a = __builtin_convertvector(lo, bf16x4), b = __builtin_convertvector(hi, bf16x4);
    *reinterpret_cast<bf16x8 *>(c) = __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
}

// Products with a short K or a small C; the order inside a step is the compiler's. A wave computes (16 TM) x (16 TN),
// WM x WN waves a block tile, which M and N are multiples of; KG such groups of waves share the tile, each taking every
// KG-th step of K, and their sums are added in LDS at the end (in group order: the result does not depend on timing).
// NST steps are in LDS; the loads of a step go out NST - 1 steps ahead. With 32 x 32 tiles a wave has one fragment of each side
// (and stores half a piece a row): what bounds a block of a long K is the panels' bytes at some 50 a cycle, and where 32 x 64
// tiles leave half of the compute units or more without one, tiles of half the size have a third less to load each:
// 256 x 512 x 7808 20.0 -> 13.8 us, 128 x 128 x 5120 12.8 -> 9.6, 256 x 384 x 1664 6.3 -> 5.2. (Fragments straight from memory, with K
// split among the waves of a block, take twice as long: sixteen rows a request.)
template <int TM, int TN, int WM, int WN, int KG, int NST, bool WIDE>
__global__ __launch_bounds__(64 * WM * WN * KG) void gemm_bf16_kernel(const uint16_t *__restrict__ A, const uint16_t *__restrict__ B,
                                                                     uint16_t *__restrict__ C, int N, int K, TileOrder order) {
    constexpr int BM = 16 * TM * WM, BN = 16 * TN * WN, NW = WM * WN, STEP = (BM + BN) * 64;
    constexpr bool PAIRS = TN % 2 == 0;
    typedef PanelLoader<BM, BN, NW, PAIRS, false, WIDE> Loader;
    static_assert(PAIRS || TN == 1, "B fragments come in pairs, or there is one");
    static_assert((KG - 1) * BM * BN * 4 <= NST * KG * STEP * 2, "the partial sums fit where the panels were");
    __shared__ __attribute__((aligned(1024))) uint16_t lds[NST * KG * STEP];
    const GemmTile t = gemm_tile(order);
    const int lane = threadIdx.x & 63, wave_all = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wave = wave_all % NW, group = wave_all / NW;
    const int wm = wave / WN, wn = wave % WN;
    const Loader load(A + size_t(t.tm) * BM * K, B + size_t(t.tn) * BN * K, K, lane, wave);
    const int steps64 = K / 64, steps = (steps64 + KG - 1) / KG;
    const bool in_last = (steps - 1) * KG + group < steps64;      // whether this group has a part of the last step
    auto issue = [&](int step, int stage) {
        if (step >= steps || (step == steps - 1 && !in_last)) return;
#pragma unroll
        for (int i = 0; i < Loader::COUNT; i++) load.issue(lds + (stage * KG + group) * STEP, step * KG + group, i);
    };
    const int ar = lane & 15, br = PAIRS ? 8 * (ar >> 2) + (ar & 3) : ar;
    int at_a[2], at_b[2];
#pragma unroll
    for (int h = 0; h < 2; h++) {
        at_a[h] = (16 * TM * wm + ar) * 64 + 8 * ((4 * h + (lane >> 4)) ^ ((ar >> 1) & 7));
        at_b[h] = (BM + 16 * TN * wn + br) * 64 + 8 * ((4 * h + (lane >> 4)) ^ (PAIRS ? ((ar >> 1) & 1) | ((ar >> 2) << 1) : (ar >> 1) & 7));
    }
    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
        for (int j = 0; j < TN; j++) acc[i][j] = f32x4{0, 0, 0, 0};
#pragma unroll
    for (int s = 0; s < NST - 1; s++) issue(s, s);
    int stage = 0, next = NST - 1;
    for (int step = 0; step < steps; step++) {
        // steps step+1 .. step+NST-2 may still be under way; near the end (where a group may lack the last one) nothing may
        if (steps - 1 - step >= NST - 2 + (KG > 1 ? 1 : 0)) wait_loads_and_meet<(NST - 2) * Loader::COUNT>();
        else wait_loads_and_meet<0>();
        issue(step + NST - 1, next);                 // over the stage every wave has just finished reading
        next = next + 1 == NST ? 0 : next + 1;
        if (step == steps - 1 && !in_last) break;
        const uint16_t *p = lds + (stage * KG + group) * STEP;
        bf16x8 fa[2][TM], fb[2][TN];
#pragma unroll
        for (int h = 0; h < 2; h++) {
#pragma unroll
            for (int j = 0; j < TN; j++) fb[h][j] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(p + at_b[h] + (j >> 1) * 2048 + (j & 1) * 256));
#pragma unroll
            for (int i = 0; i < TM; i++) fa[h][i] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(p + at_a[h] + i * 1024));
        }
#pragma unroll
        for (int h = 0; h < 2; h++)
#pragma unroll
            for (int i = 0; i < TM; i++)
#pragma unroll
                for (int j = 0; j < TN; j++) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[h][j], fa[h][i], acc[i][j], 0, 0, 0);
        stage = stage + 1 == NST ? 0 : stage + 1;
    }
    if constexpr (KG > 1) {
        f32x4 *part = reinterpret_cast<f32x4 *>(lds);
        __syncthreads();
        if (group > 0) {
#pragma unroll
            for (int i = 0; i < TM * TN; i++) part[(((group - 1) * NW + wave) * TM * TN + i) * 64 + lane] = acc[i / TN][i % TN];
        }
        __syncthreads();
        if (group > 0) return;
#pragma unroll
        for (int g = 0; g < KG - 1; g++)
#pragma unroll
            for (int i = 0; i < TM * TN; i++) acc[i / TN][i % TN] += part[((g * NW + wave) * TM * TN + i) * 64 + lane];
    }
    uint16_t *c = C + (size_t(t.tm) * BM + wm * 16 * TM + ar) * N + size_t(t.tn) * BN + wn * 16 * TN + (PAIRS ? 8 : 4) * (lane >> 4);
#pragma unroll
    for (int i = 0; i < TM; i++) {
        if constexpr (!PAIRS) *reinterpret_cast<bf16x4 *>(c + size_t(16 * i) * N) = __builtin_convertvector(acc[i][0], bf16x4);
        else
#pragma unroll
            for (int j = 0; j < TN; j += 2) store_columns(c + size_t(16 * i) * N + 16 * j, acc[i][j], acc[i][j + 1]);
    }
}

template <class F, int... I>
__device__ __forceinline__ void for_each_of(F f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }

// The other products: WM x WN waves, each computing (16 TM) x (16 TN) of the block's tile, ONE wave per SIMD or two. Nothing
// hides a wait but the wave's own order, so the order is fixed by hand: a step of 64 K values is 2 TM TN MFMAs, and
// between them, at the places given below, go the 2 (TM + TN) fragment reads and the panel loads. The fragments of one half
// of a step (32 K values) are read under the MFMAs of the half before, READS a MFMA or (negative) one in -READS MFMAs; the
// panel loads go out one every LOAD_EVERY MFMAs (64 bytes a cycle is what a compute unit takes, 44 to 58 what it was
// seen to take). STAGES steps are in LDS:
//   two     once every wave has read its second half's fragments of this step the stage is free, and the loads of step + 2
//           into it start; three quarters into the step the loads of step + 1 have landed for all (those of step + 2 issued
//           so far may be under way), and the fragments of its first half are read under the rest of this step;
//   more    both in one meeting at the beginning of the second half. The loads that this frees the stage for go on
//           into the next step, up to its meeting.
// A load thus has most of a step and more before it is waited for. Tiles of more than 128 x 128 per SIMD pair name the
// accumulators as AGPRs in the MFMA's own operands: left to itself the compiler moves them to and fro between the two
// register files inside the loop.
// MFMAs go to and fro along B's fragments, so that two in a row always share an operand (0.3 % at 8192^3).
// M is at least BM and N at least BN, both multiples of 32. The last tile of a row or column ends at the edge of C: it
// starts inside the one before it where BM or BN does not divide, and both write the same bits there.
//
// What bounds it: the power, with 256 x 256 tiles (1.76 GHz at 92 % of the matrix pipe's cycles in the loop; 8192^3 in
// 0.69 to 0.72 ms = 1590 to 1530 TFLOP/s, where one 32x32x16 kernel with panels through registers took 1.07), and towards small tiles
// more and more what a wave issues between its MFMAs and the panel loads (BM + BN rows a step): 128 x 128 takes 820 cycles a step,
// of which the MFMAs are 512 and the loads at 58 bytes a cycle 565. Four waves of 64 x 64 instead of sixteen of 32 x 32
// and a hand-made order made of 1024 x 3072 x 768 9.8 -> 7.4 us, launched in a row.
template <int WM, int WN, int TM, int TN, int STAGES, int READS, int LOAD_EVERY, bool WIDE>
__device__ __forceinline__ void gemm_bf16_tile(const uint16_t *__restrict__ A, const uint16_t *__restrict__ B, uint16_t *__restrict__ C, int M, int N, int K,
                                               const TileOrder &order) {
    constexpr int NW = WM * WN, BM = 16 * TM * WM, BN = 16 * TN * WN, STEP = (BM + BN) * 64, FRAGS = TM + TN, HALF = TM * TN;
    constexpr bool NAMED = TM * TN > 32, TWO = STAGES == 2;
    typedef PanelLoader<BM, BN, NW, true, !NAMED, WIDE> Loader;
    constexpr int COUNT = Loader::COUNT;
    static_assert(TN % 2 == 0 && STAGES >= 2, "B fragments come in pairs");
    // fragment i of a half is read behind MFMA at_read(i) of the half before it (of what is left of that behind the second meeting)
    constexpr int PACE = READS > 0 ? READS : 1, AT_ONCE = READS > 0 ? 1 : -READS;
    constexpr int READ_SPAN = (FRAGS + AT_ONCE - 1) / AT_ONCE * PACE;
    constexpr int FREE_AT = TWO ? (READ_SPAN + 8 < HALF ? READ_SPAN + 8 : READ_SPAN + 4 < HALF ? READ_SPAN + 4 : HALF) : HALF + 2;
    constexpr int LANDED_AT = TWO ? HALF + HALF / 2 : HALF + 2;
    constexpr int FITTING = (2 * HALF - FREE_AT + LOAD_EVERY - 1) / LOAD_EVERY;       // loads that go out in the step that frees their stage
    constexpr int NOW = TWO || FITTING > COUNT ? COUNT : FITTING;
    constexpr int GONE = (LANDED_AT - FREE_AT + LOAD_EVERY - 1) / LOAD_EVERY;         // two stages: those of them out at the second meeting
    constexpr int UNDER_WAY = TWO ? (GONE < COUNT ? GONE : COUNT) : (STAGES - 2) * COUNT;
    static_assert(READ_SPAN <= HALF && FREE_AT <= HALF + 2 && LANDED_AT < 2 * HALF, "the reads of a half lie inside the half before");
    static_assert(TWO || FREE_AT + (COUNT - 1) * LOAD_EVERY - 2 * HALF < LANDED_AT, "a step's loads are out before the next one's");
    __shared__ __attribute__((aligned(1024))) uint16_t lds[STAGES * STEP];
    const GemmTile t = gemm_tile(order);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wm = wave / WN, wn = wave % WN;
    const int row = min(t.tm * BM, M - BM), col = min(t.tn * BN, N - BN);
    const Loader load(A + size_t(row) * K, B + size_t(col) * K, K, lane, wave);
    const int ar = lane & 15, br = 8 * (ar >> 2) + (ar & 3);
    int at_a[2], at_b[2];
#pragma unroll
    for (int h = 0; h < 2; h++) {
        at_a[h] = (16 * TM * wm + ar) * 64 + 8 * ((4 * h + (lane >> 4)) ^ ((ar >> 1) & 7));
        at_b[h] = (BM + 16 * TN * wn + br) * 64 + 8 * ((4 * h + (lane >> 4)) ^ (((ar >> 1) & 1) | ((ar >> 2) << 1)));
    }
    bf16x8 frag[2][FRAGS];      // [half of the step]: B fragments first, then A
    auto read = [&](int half, int stage, int i) {
        const uint16_t *p = lds + stage * STEP + (i < TN ? at_b[half] + (i >> 1) * 2048 + (i & 1) * 256 : at_a[half] + (i - TN) * 1024);
        frag[half][i] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(p));
    };
    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
        for (int j = 0; j < TN; j++) acc[i][j] = f32x4{0, 0, 0, 0};
    const int steps = K / 64;
    // Past the end the last step is loaded again, into a stage nothing reads.
#pragma unroll
    for (int s = 0; s < STAGES; s++)
#pragma unroll
        for (int i = 0; i < (s == STAGES - 1 ? NOW : COUNT); i++) load.issue(lds + s * STEP, s < steps ? s : steps - 1, i);
    wait_loads_and_meet<(STAGES - 2) * COUNT + NOW>();
#pragma unroll
    for (int i = 0; i < FRAGS; i++) read(0, 0, i);
    if constexpr (NAMED) {
        // The accumulators are set by ordinary instructions and read by the asm below, for which the compiler inserts no wait
        // states: they are in their registers before the fence, which nothing moves across.
#pragma unroll
        for (int i = 0; i < TM; i++)
#pragma unroll
            for (int j = 0; j < TN; j++) asm volatile("" : "+a"(acc[i][j]));
        asm volatile("s_nop 7");
    }
    __builtin_amdgcn_sched_barrier(0);
    int in_turn = 0;
    for (int step = 0; step < steps; step++) {
        const int stage = TWO ? step & 1 : in_turn, next = TWO ? stage ^ 1 : stage + 1 == STAGES ? 0 : stage + 1;
        const int before = stage == 0 ? STAGES - 1 : stage - 1;
        const int ahead = step + STAGES < steps ? step + STAGES : steps - 1, late = step + STAGES - 1 < steps ? step + STAGES - 1 : steps - 1;
        for_each_of([&](auto index) {
            constexpr int at = index, half = at / HALF, i = at % HALF / TN, j = i & 1 ? TN - 1 - at % TN : at % TN;
            if constexpr (TWO && at == FREE_AT) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            if constexpr (at == LANDED_AT && TWO) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(UNDER_WAY) : "memory");
            if constexpr (at == LANDED_AT && !TWO) wait_loads_and_meet<UNDER_WAY>();
            if constexpr (NAMED) asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc[i][j]) : "v"(frag[half][j]), "v"(frag[half][TN + i]));
            else acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(frag[half][j], frag[half][TN + i], acc[i][j], 0, 0, 0);
#pragma unroll
            for (int q = 0; q < AT_ONCE; q++) {
                if (at < HALF && at % PACE == 0 && at / PACE * AT_ONCE + q < FRAGS) read(1, stage, at / PACE * AT_ONCE + q);
                if (at >= LANDED_AT && (at - LANDED_AT) % PACE == 0 && (at - LANDED_AT) / PACE * AT_ONCE + q < FRAGS)
                    read(0, next, (at - LANDED_AT) / PACE * AT_ONCE + q);
            }
            if constexpr (at >= FREE_AT && (at - FREE_AT) % LOAD_EVERY == 0 && (at - FREE_AT) / LOAD_EVERY < COUNT)
                load.issue(lds + stage * STEP, ahead, (at - FREE_AT) / LOAD_EVERY);
            constexpr int since = at + 2 * HALF - FREE_AT;      // MFMAs since the stage of the step before was free
            if constexpr (NOW < COUNT && at < LANDED_AT && since % LOAD_EVERY == 0 && since / LOAD_EVERY < COUNT)
                load.issue(lds + before * STEP, late, since / LOAD_EVERY);
            __builtin_amdgcn_sched_barrier(0);
        }, std::make_integer_sequence<int, 2 * HALF>{});
        // what there was no MFMA left for
#pragma unroll
        for (int i = FITTING; i < NOW; i++) load.issue(lds + stage * STEP, ahead, i);
#pragma unroll
        for (int i = (2 * HALF - LANDED_AT + PACE - 1) / PACE * AT_ONCE; i < FRAGS; i++) read(0, next, i);
        __builtin_amdgcn_sched_barrier(0);
        in_turn = next;
    }
    // the last MFMAs' results are readable, and no load to LDS outlives the block
    asm volatile("s_nop 15\n\ts_nop 15\n\ts_waitcnt vmcnt(0)" ::: "memory");
    uint16_t *c = C + size_t(row + wm * 16 * TM + ar) * N + col + wn * 16 * TN + 8 * (lane >> 4);
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
        for (int j = 0; j < TN; j += 2) {
            // in their registers up to here: copied out all at once they would spill
            if constexpr (NAMED) asm volatile("" : "+a"(acc[i][j]), "+a"(acc[i][j + 1]));
            store_columns(c + size_t(16 * i) * N + 16 * j, acc[i][j], acc[i][j + 1]);
            __builtin_amdgcn_sched_barrier(0);
        }
}

// TOGETHER blocks share a compute unit. The bodies are the device's only: the host's pass needs no more than the names.
template <int TOGETHER, int WM, int WN, int TM, int TN, int STAGES, int READS, int LOAD_EVERY, bool WIDE>
__global__ __launch_bounds__(256, TOGETHER) void gemm_bf16_tile_kernel(const uint16_t *__restrict__ A, const uint16_t *__restrict__ B,
                                                                      uint16_t *__restrict__ C, int M, int N, int K, TileOrder order) {
#if defined(__HIP_DEVICE_COMPILE__)
    gemm_bf16_tile<WM, WN, TM, TN, STAGES, READS, LOAD_EVERY, WIDE>(A, B, C, M, N, K, order);
#endif
}
template <bool WIDE>
__global__ __launch_bounds__(256) void gemm_bf16_256_kernel(const uint16_t *__restrict__ A, const uint16_t *__restrict__ B, uint16_t *__restrict__ C, int M,
                                                           int N, int K, TileOrder order) {
#if defined(__HIP_DEVICE_COMPILE__)
    gemm_bf16_tile<2, 2, 8, 8, 2, 2, 4, WIDE>(A, B, C, M, N, K, order);
#endif
}

template <bool WIDE>
void launch_gemm(const uint16_t *a, const uint16_t *b, uint16_t *c, int m, int n, int k, hipStream_t stream) {
    const int choice = gemm_form(m, n, k);
    const GemmForm &form = kGemmForms[choice];
    const unsigned tm = form.tiles_m(m), tn = form.tiles_n(n);
    // `simple`: the kernels whose order is the compiler's; `by_xcd`: see TileOrder
    auto simple = [&](auto kernel, bool by_xcd) {
        hipLaunchKernelGGL(kernel, dim3(tm * tn), dim3(form.threads), 0, stream, a, b, c, n, k, TileOrder(tm, tn, by_xcd));
    };
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(tm * tn), dim3(form.threads), 0, stream, a, b, c, m, n, k, TileOrder(tm, tn, true));
    };
    switch (choice) {
        case 0: go(gemm_bf16_256_kernel<WIDE>); break;
        case 1: go(gemm_bf16_tile_kernel<1, 2, 2, 7, 8, 2, 2, 4, WIDE>); break;
        case 2: go(gemm_bf16_tile_kernel<1, 2, 2, 8, 6, 2, 2, 4, WIDE>); break;
        case 3: go(gemm_bf16_tile_kernel<1, 2, 2, 5, 8, 3, 2, 4, WIDE>); break;
        case 4: go(gemm_bf16_tile_kernel<2, 2, 2, 6, 4, 2, 1, 2, WIDE>); break;
        case 5: go(gemm_bf16_tile_kernel<1, 2, 2, 5, 4, 3, 1, 4, WIDE>); break;
        case 6: go(gemm_bf16_tile_kernel<1, 2, 2, 4, 4, 3, 1, 4, WIDE>); break;
        case 7: if constexpr (!WIDE) go(gemm_bf16_tile_kernel<2, 2, 2, 4, 4, 2, -2, 1, false>); break;
        case 8: go(gemm_bf16_tile_kernel<1, 4, 1, 2, 6, 3, 1, 3, WIDE>); break;
        case 9: go(gemm_bf16_tile_kernel<2, 2, 2, 2, 4, 3, 1, 2, WIDE>); break;
        case 10: go(gemm_bf16_tile_kernel<2, 2, 2, 3, 2, 4, -2, 1, WIDE>); break;
        case 11: go(gemm_bf16_tile_kernel<2, 2, 2, 2, 2, 4, -2, 1, WIDE>); break;
        case 12: if constexpr (!WIDE) go(gemm_bf16_tile_kernel<3, 2, 2, 2, 2, 3, -2, 1, false>); break;
        case 13: simple(gemm_bf16_kernel<1, 2, 2, 2, 4, 3, WIDE>, true); break;
        case 14: simple(gemm_bf16_kernel<1, 1, 2, 2, 4, 3, WIDE>, true); break;
        case 15: if constexpr (!WIDE) simple(gemm_bf16_kernel<4, 4, 2, 2, 1, 2, false>, false); break;
        // up to K = 192
        case 16: if constexpr (!WIDE) simple(gemm_bf16_kernel<2, 2, 2, 2, 1, 3, false>, false); break;
        case 17: if constexpr (!WIDE) simple(gemm_bf16_kernel<2, 4, 2, 2, 1, 2, false>, false); break;
        default: if constexpr (!WIDE) simple(gemm_bf16_kernel<2, 4, 4, 2, 1, 2, false>, true); break;
    }
}

unsigned blocks_for(uint64_t n, unsigned per_block) {
    uint64_t b = (n + per_block - 1) / per_block;
    const uint64_t cap = 256 * 16;   // 16 resident blocks' worth per CU; the kernels are grid-stride
    return unsigned(b < 1 ? 1 : (b > cap ? cap : b));
}

int hip_rc() { return hipGetLastError() == hipSuccess ? 0 : -4; }

}  // namespace

extern "C" {

int proxy_gemm_bf16(const void *a, const void *b, void *c, int32_t m, int32_t n, int32_t k, void *stream) {
    if (!a || !b || !c || m <= 0 || n <= 0 || k <= 0 || m % 128 || n % 128 || k % 64) return -1;
    if ((uint64_t(a) | uint64_t(b) | uint64_t(c)) & 15) return -1;
    const auto launch = gemm_wide(k) ? launch_gemm<true> : launch_gemm<false>;
    launch(static_cast<const uint16_t *>(a), static_cast<const uint16_t *>(b), static_cast<uint16_t *>(c), m, n, k, static_cast<hipStream_t>(stream));
    return hip_rc();
}

int proxy_fill_state(void *p, void *master, void *m, void *v, uint64_t numel, uint64_t seed, uint64_t tensor, void *stream) {
    if (!p || !master || !m || !v || numel == 0) return -1;
    hipLaunchKernelGGL(fill_state_kernel, dim3(blocks_for(numel, 256)), dim3(256), 0, static_cast<hipStream_t>(stream),
                       static_cast<uint16_t *>(p), static_cast<float *>(master), static_cast<float *>(m), static_cast<float *>(v), numel,
                       stream_key(seed, tensor, 0), stream_key(seed, tensor, 1), stream_key(seed, tensor, 2));
    return hip_rc();
}

int proxy_adam_step(void *p, void *master, void *m, void *v, uint64_t numel, uint64_t seed, uint64_t tensor, uint64_t step, float lr,
                    float beta1, float beta2, float eps, void *stream) {
    if (!p || !master || !m || !v || numel == 0 || step == 0) return -1;
    if (((uint64_t(master) | uint64_t(m) | uint64_t(v)) & 15) || (uint64_t(p) & 7)) return -1;
    AdamArgs a;
    a.lr = lr; a.beta1 = beta1; a.beta2 = beta2; a.eps = eps;
    a.inv_bc1 = float(1.0 / (1.0 - pow(double(beta1), double(step))));
    a.inv_bc2 = float(1.0 / (1.0 - pow(double(beta2), double(step))));
    const uint64_t quads = (numel + 3) / 4, most = 1ull << 31;     // a grid has fewer than 2^32 work-items
    for (uint64_t first = 0; first < quads; first += most) {
        const unsigned blocks = unsigned((std::min(quads - first, most) + 63) / 64);
        hipLaunchKernelGGL(adam_kernel, dim3(blocks), dim3(64), blocks > kAdamFreeBlocks ? kAdamLds : 0, static_cast<hipStream_t>(stream),
                           static_cast<uint16_t *>(p), static_cast<float *>(master), static_cast<float *>(m), static_cast<float *>(v), numel, first,
                           stream_key(seed + step, tensor, 3), a);
    }
    return hip_rc();
}

int proxy_fill_words(void *w, uint64_t n, uint64_t seed, void *stream) {
    if (!w || n == 0 || (uint64_t(w) & 3)) return -1;
    hipLaunchKernelGGL(fill_words_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, static_cast<hipStream_t>(stream), static_cast<uint32_t *>(w), n,
                       stream_key(seed, 0, 0));
    return hip_rc();
}

int proxy_mutate_words(void *w, uint64_t n, uint64_t step, void *stream) {
    if (!w || n == 0 || (uint64_t(w) & 3)) return -1;
    hipLaunchKernelGGL(mutate_words_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, static_cast<hipStream_t>(stream), static_cast<uint32_t *>(w), n,
                       uint32_t(step));
    return hip_rc();
}

int proxy_devcopy(void *dst, const void *src, uint64_t nbytes, void *stream) {
    if (!dst || !src || nbytes == 0 || (nbytes & 15) || ((uint64_t(dst) | uint64_t(src)) & 15)) return -1;
    const uint64_t n16 = nbytes >> 4, most = 1ull << 31;     // a grid has fewer than 2^32 work-items
    for (uint64_t first = 0; first < n16; first += most) {
        const uint64_t n = std::min(n16 - first, most);
        hipLaunchKernelGGL(devcopy_kernel, dim3(unsigned((n + 63) / 64)), dim3(64), 0, static_cast<hipStream_t>(stream),
                           static_cast<u32x4 *>(dst) + first, static_cast<const u32x4 *>(src) + first, n);
    }
    return hip_rc();
}

#define PROXY_TRY(expr) do { if ((expr) != hipSuccess) { (void)hipGetLastError(); return -4; } } while (0)

int proxy_device_alloc(uint64_t nbytes, void **out) {
    if (!out || nbytes == 0) return -1;
    PROXY_TRY(hipMalloc(out, nbytes));
    return 0;
}
int proxy_device_free(void *dev) { if (!dev) return -1; PROXY_TRY(hipFree(dev)); return 0; }
int proxy_host_alloc_pinned(uint64_t nbytes, void **out) {
    if (!out || nbytes == 0) return -1;
    PROXY_TRY(hipHostMalloc(out, nbytes, hipHostMallocDefault));
    for (uint64_t o = 0; o < nbytes; o += 4096) static_cast<volatile char *>(*out)[o] = 0;
    return 0;
}
int proxy_host_free_pinned(void *host) { if (!host) return -1; PROXY_TRY(hipHostFree(host)); return 0; }
int proxy_copy_h2d(void *dst, const void *src, uint64_t n) { if (!dst || !src) return -1; if (n) PROXY_TRY(hipMemcpy(dst, src, n, hipMemcpyHostToDevice)); return 0; }
int proxy_copy_d2h(void *dst, const void *src, uint64_t n) { if (!dst || !src) return -1; if (n) PROXY_TRY(hipMemcpy(dst, src, n, hipMemcpyDeviceToHost)); return 0; }
int proxy_copy_d2d_async(void *dst, const void *src, uint64_t n, void *stream) {
    if (!dst || !src) return -1;
    if (n) PROXY_TRY(hipMemcpyAsync(dst, src, n, hipMemcpyDeviceToDevice, static_cast<hipStream_t>(stream)));
    return 0;
}
int proxy_copy_pinned_async(void *dst, const void *src, uint64_t n, int32_t to_host, void *stream) {
    if (!dst || !src) return -1;
    if (n) PROXY_TRY(hipMemcpyAsync(dst, src, n, to_host ? hipMemcpyDeviceToHost : hipMemcpyHostToDevice, static_cast<hipStream_t>(stream)));
    return 0;
}
int proxy_device_fill_async(void *dev, int32_t byte, uint64_t n, void *stream) {
    if (!dev) return -1;
    if (n) PROXY_TRY(hipMemsetAsync(dev, byte, n, static_cast<hipStream_t>(stream)));
    return 0;
}
int proxy_stream_synchronize(void *stream) { PROXY_TRY(hipStreamSynchronize(static_cast<hipStream_t>(stream))); return 0; }
int proxy_device_synchronize(void) { PROXY_TRY(hipDeviceSynchronize()); return 0; }
int proxy_event_create(void **out) { if (!out) return -1; hipEvent_t e; PROXY_TRY(hipEventCreate(&e)); *out = e; return 0; }
int proxy_event_destroy(void *e) { if (!e) return -1; PROXY_TRY(hipEventDestroy(static_cast<hipEvent_t>(e))); return 0; }
int proxy_event_record(void *e, void *stream) { if (!e) return -1; PROXY_TRY(hipEventRecord(static_cast<hipEvent_t>(e), static_cast<hipStream_t>(stream))); return 0; }
int proxy_event_synchronize(void *e) { if (!e) return -1; PROXY_TRY(hipEventSynchronize(static_cast<hipEvent_t>(e))); return 0; }
int proxy_event_elapsed_ms(void *a, void *b, float *ms) {
    if (!a || !b || !ms) return -1;
    PROXY_TRY(hipEventElapsedTime(ms, static_cast<hipEvent_t>(a), static_cast<hipEvent_t>(b)));
    return 0;
}
int proxy_device_info(char *name, uint64_t cap, int32_t *cus, uint64_t *total, uint64_t *free_, int32_t *ver) {
    int dev = 0;
    PROXY_TRY(hipGetDevice(&dev));
    hipDeviceProp_t p;
    PROXY_TRY(hipGetDeviceProperties(&p, dev));
    if (name && cap) { snprintf(name, cap, "%s (%s)", p.name, p.gcnArchName); }
    if (cus) *cus = p.multiProcessorCount;
    size_t f = 0, t = 0;
    PROXY_TRY(hipMemGetInfo(&f, &t));
    if (total) *total = t;
    if (free_) *free_ = f;
    int v = 0;
    PROXY_TRY(hipRuntimeGetVersion(&v));
    if (ver) *ver = v;
    return 0;
}

int proxy_stream_create(void **out) {
    if (!out) return -1;
    hipStream_t s = nullptr;
    if (hipStreamCreateWithFlags(&s, hipStreamNonBlocking) != hipSuccess) return -4;
    *out = s;
    return 0;
}

int proxy_stream_destroy(void *stream) {
    if (!stream) return -1;
    return hipStreamDestroy(static_cast<hipStream_t>(stream)) == hipSuccess ? 0 : -4;
}

}  // extern "C"
