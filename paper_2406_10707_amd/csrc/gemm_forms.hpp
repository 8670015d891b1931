// Which kernel and tile the training proxy's GEMM takes for a product. Host code that needs no HIP, so that a test can ask it.
#pragma once
#include <math.h>
#include <stdint.h>

namespace dsllm {

// Which kernel and tile: the one of these that is expected to be done first. Up to K = 192 it is the first lines of gemm_form
// that decide, as a product is then little more than a launch and the stores of C (the hand-made order's prologue costs 0.5 us
// more than the other kernel's: 2432 x 4992 x 64 8.8 us against 10.0). 64 x 64 tiles as long as they are all under way at once,
// three to a unit. Then what counts is how many rounds of blocks there are: a round of 64 x 128 tiles, three to a unit, is
// three quarters of the data of one of 128 x 128, two to a unit, and takes about 0.8 of its time. Four waves a 128 x 128 tile in a single round
// or with K = 64; else eight, in the XCDs' order, as panels are then read again by other rounds. Over 225 products
// 2.9 % faster than 64 x 64, sixteen-wave 128 x 128 and four-wave 128 x 128 tiles by their number alone, and none slower:
//   896 x 3456 x 64 4.76 -> 4.33         640 x 6784 x 64 5.76 -> 4.86      7040 x 1280 x 128 9.4 -> 8.2
//   1792 x 7808 x 192 14.2 -> 12.8       3456 x 7808 x 192 26.1 -> 20.2
//
// What a form is expected to take, in us: `start`, and then for the compute unit with the most blocks, which takes them in
// rounds of up to `together`, block[n - 1] + step[n - 1] * (K / 64) for every round of n; and for all blocks together, as a
// full card clocks lower and shares memory, (spread_block + spread_step * (K / 64)) * blocks / 256. The figures are fitted to times
// of every form on 560 products on an MI355X, M and N multiples of 128 up to 8192 and K of 64 up to 8192, each spread over the
// logarithm of its range (32 x 32: on 75 of them): 2 to 3 % off in the mean, 4 to 9 % at the ninth decile. The choice by them is 1.1 % slower in the
// mean than the best form for each product. Against a rule on the number of tiles over two 128 x 128, two 64 x 64, one 32 x 64 kernel and
// 256 x 256 where both sizes are its multiples, 300 other products of these ranges take 16 % less time in the mean, and 40 with K of 8192 to
// 131072, for which nothing was fitted, 19 % (none of either more than 2 % longer). Where the rule lost most:
//   1152 x 7808 x 53568 1511 -> 747 us
//   6272 x 7808 x 6592 686 -> 479        sizes not multiples of 256, formerly 128 x 128 for all
//   1920 x 7936 x 3456 127 -> 76
//   768 x 5632 x 3392 46 -> 34           a few 128 x 128 tiles more than there are units
//   384 x 5248 x 960 12.1 -> 6.9
//   1024 x 3072 x 768 9.8 -> 7.4         fewer 128 x 128 tiles than units: 128 x 96 fills them
// One product was found that loses more than that: 7040 x 2688 x 256 17.8 -> 18.5 (of 400 more with K of 256 to 512 none).
// WIDE once a panel of 256 rows passes 2 GiB (the offsets of a buffer load are 32 bits wide). The choice is the same there, but for
// three forms, which aren't built for it: two were never chosen, and 128 x 128 by 2 for ten pairs of sizes among those whose
// operands fit the card (20608..21760 x 384; 20608 x 384 takes 122 to 127 ms with it and 123 to 130 without).
struct GemmForm {
    const char *name;        // tile; "by n": n blocks share a compute unit
    int rows, cols, threads, together;
    bool wide;               // built for K above 2^22 too
    float start, block[3], step[3], spread_block, spread_step;

    unsigned tiles_m(int m) const { return (unsigned(m) + unsigned(rows) - 1) / unsigned(rows); }
    unsigned tiles_n(int n) const { return (unsigned(n) + unsigned(cols) - 1) / unsigned(cols); }
    float expected(int m, int n, int k) const {
        if (m < rows || n < cols) return INFINITY;
        const float steps = float(k / 64), blocks = float(m / rows + (m % rows != 0)) * float(n / cols + (n % cols != 0));
        const float per_unit = ceilf(blocks / 256), rounds = floorf(per_unit / float(together));
        const int rest = int(per_unit - rounds * float(together));
        float us = start + rounds * (block[together - 1] + step[together - 1] * steps) + (spread_block + spread_step * steps) * blocks / 256;
        if (rest) us += block[rest - 1] + step[rest - 1] * steps;
        return us;
    }
};
constexpr GemmForm kGemmForms[] = {     // in the order of launch_gemm's switch
    {"256x256", 256, 256, 256, 1, true, 2.43f, {3.90f, 0.00f, 0.00f}, {0.9122f, 0.0000f, 0.0000f}, 4.56f, 0.2758f},
    {"224x256", 224, 256, 256, 1, true, 1.94f, {3.93f, 0.00f, 0.00f}, {0.7984f, 0.0000f, 0.0000f}, 3.95f, 0.2545f},
    {"256x192", 256, 192, 256, 1, true, 1.71f, {3.74f, 0.00f, 0.00f}, {0.6975f, 0.0000f, 0.0000f}, 3.20f, 0.2218f},
    {"160x256", 160, 256, 256, 1, true, 1.24f, {3.91f, 0.00f, 0.00f}, {0.5994f, 0.0000f, 0.0000f}, 2.76f, 0.1911f},
    {"192x128 by 2", 192, 128, 256, 2, true, 2.94f, {1.14f, 2.09f, 0.00f}, {0.4599f, 0.8657f, 0.0000f}, 1.45f, 0.1007f},
    {"160x128", 160, 128, 256, 1, true, 1.35f, {2.72f, 0.00f, 0.00f}, {0.3502f, 0.0000f, 0.0000f}, 0.69f, 0.1319f},
    {"128x128", 128, 128, 256, 1, true, 1.26f, {2.39f, 0.00f, 0.00f}, {0.3033f, 0.0000f, 0.0000f}, 0.39f, 0.1069f},
    {"128x128 by 2", 128, 128, 256, 2, false, 2.56f, {0.84f, 1.66f, 0.00f}, {0.3865f, 0.6772f, 0.0000f}, 0.94f, 0.0625f},
    {"128x96", 128, 96, 256, 1, true, 1.28f, {1.93f, 0.00f, 0.00f}, {0.2641f, 0.0000f, 0.0000f}, 0.25f, 0.0856f},
    {"64x128 by 2", 64, 128, 256, 2, true, 1.75f, {1.02f, 1.53f, 0.00f}, {0.2244f, 0.4022f, 0.0000f}, 0.20f, 0.0705f},
    {"96x64 by 2", 96, 64, 256, 2, true, 1.73f, {1.01f, 1.32f, 0.00f}, {0.1853f, 0.3621f, 0.0000f}, 0.23f, 0.0407f},
    {"64x64 by 2", 64, 64, 256, 2, true, 1.80f, {0.67f, 0.89f, 0.00f}, {0.1494f, 0.2870f, 0.0000f}, 0.18f, 0.0281f},
    {"64x64 by 3", 64, 64, 256, 3, false, 2.07f, {0.17f, 0.58f, 1.24f}, {0.1521f, 0.2266f, 0.3086f}, 0.00f, 0.0740f},
    {"32x64 K/4", 32, 64, 1024, 1, true, 1.37f, {1.66f, 0.00f, 0.00f}, {0.1244f, 0.0000f, 0.0000f}, 0.17f, 0.0134f},
    {"32x32 K/4", 32, 32, 1024, 1, true, 1.25f, {1.74f, 0.00f, 0.00f}, {0.0820f, 0.0000f, 0.0000f}, 0.08f, 0.0071f},
    {"128x128 compiled", 128, 128, 256, 2, false, 2.24f, {0.55f, 1.81f, 0.00f}, {0.5691f, 0.6548f, 0.0000f}, 0.76f, 0.1264f},
    // up to K = 192 only: no model
    {"64x64 short", 64, 64, 256, 3, false, INFINITY, {}, {}, 0, 0},
    {"64x128 short", 64, 128, 256, 3, false, INFINITY, {}, {}, 0, 0},
    {"128x128 short, eight waves", 128, 128, 512, 2, false, INFINITY, {}, {}, 0, 0},
};
constexpr int kModelledForms = 16;

inline bool gemm_wide(int k) { return k > (1 << 22); }

// M and N multiples of 128, K of 64
inline int gemm_form(int m, int n, int k) {
    if (k <= 192) {
        const int64_t n64 = int64_t(m / 64) * (n / 64);
        const int64_t rounds_of_half = (n64 / 2 + 3 * 256 - 1) / (3 * 256), rounds_of_128 = (n64 / 4 + 2 * 256 - 1) / (2 * 256);
        if (n64 <= 3 * 256) return 16;
        if (4 * rounds_of_half <= 5 * rounds_of_128) return 17;
        // (eight waves a tile only where the grid has fewer than 2^32 work-items, as it must: below 2^37 elements of C)
        return k == 64 || rounds_of_128 == 1 || n64 / 4 >= 1 << 23 ? 15 : 18;
    }
    int best = 0;
    float us = kGemmForms[0].expected(m, n, k);
    for (int f = 1; f < kModelledForms; f++) {
        if (gemm_wide(k) && !kGemmForms[f].wide) continue;
        const float t = kGemmForms[f].expected(m, n, k);
        if (t < us) { us = t; best = f; }
    }
    return best;
}

}  // namespace dsllm
