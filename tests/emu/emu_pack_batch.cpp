// Host emulation of pack_batch_kernel under AddressSanitizer (see hip/hip_runtime.h here): the image of random tensor
// lists must be the concatenation of the tensors, each padded with zeros to 4 KiB, and the one the tile-table path
// (build_tiles.hpp + pack_kernel) writes. Compiled with a small DSLLM_PACK_BATCH_PAGES, so that batches end for
// either reason (pieces, pages) and tensors are split across launches. Every tensor sits in a buffer of exactly the
// 16-byte lines it touches, so a read past them is reported.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "../../paper_2406_10707_amd/csrc/pack_kernels.hip"
#include "../../paper_2406_10707_amd/csrc/plan.hpp"
#include "build_tiles.hpp"

#ifndef EMU_BATCH
#define EMU_BATCH PackBatch
#define EMU_PIECES kPackBatch
#endif

thread_local dim3 threadIdx, blockIdx, blockDim, gridDim;
ssize_t emu_pwrite(int, const void *, size_t, off_t) { return -1; }   // no file is written here

int main(int argc, char **argv) {
    using namespace dsllm;
    uint64_t state = argc > 1 ? strtoull(argv[1], nullptr, 10) : 1;
    const int n = argc > 2 ? atoi(argv[2]) : 100;
    const uint64_t limit = argc > 3 ? strtoull(argv[3], nullptr, 10) : 20000;   // largest random size
    auto rnd = [&] { state = state * 6364136223846793005ull + 1442695040888963407ull; return state >> 33; };
    struct Piece { uint8_t *base; uint64_t lead, nbytes; };
    std::vector<Piece> ts;
    uint64_t data = 0, tiles = 0;
    for (int k = 0; k < n; k++) {
        static const uint64_t edge[] = {1, 15, 16, 17, 1023, 1024, 1025, 4080, 4081, 4095, 4096, 4097, 8191, 8192, 8193, 32768, 32769};
        Piece t;
        t.lead = k < 16 ? uint64_t(k) : rnd() % 16;
        t.nbytes = rnd() % 2 ? edge[rnd() % 17] : 1 + rnd() % limit;
        const uint64_t hull = (t.lead + t.nbytes + 15) / 16 * 16;
        t.base = static_cast<uint8_t *>(aligned_alloc(16, hull));
        for (uint64_t i = 0; i < hull; i++) t.base[i] = uint8_t(rnd() | 1);
        ts.push_back(t);
        tiles += tiles_of(data, t.nbytes, kTileBytes);
        data += (t.nbytes + 4095) / 4096 * 4096;
    }
    std::vector<uint8_t> want(data, 0);
    uint64_t off = 0;
    for (auto &t : ts) { memcpy(&want[off], t.base + t.lead, t.nbytes); off += (t.nbytes + 4095) / 4096 * 4096; }

    uint8_t *image = static_cast<uint8_t *>(aligned_alloc(4096, data));
    memset(image, 0xCC, data);
    EMU_BATCH bt;
    bt.clear();
    uint8_t *at = image;
    int launches = 0, full_pieces = 0, full_pages = 0;
    auto launch = [&] {
        full_pieces += bt.count == uint32_t(EMU_PIECES);
        full_pages += bt.first_page[bt.count] == kPackBatchPages;
        launch_pack_batch(bt, at, nullptr);
        at += kPackPage * bt.first_page[bt.count];
        bt.clear();
        launches++;
    };
    launch();   // a batch without pieces touches nothing
    for (auto &t : ts)
        for (uint64_t a = uint64_t(t.base + t.lead), left = t.nbytes; left;) {
            const uint64_t took = bt.add(a, left);
            if (took == 0 || took > left || bt.src(bt.count - 1) != a || bt.pad(bt.count - 1) >= kPackPage) { printf("add() took %llu of %llu\n", (unsigned long long)took, (unsigned long long)left); return 1; }
            a += took; left -= took;
            if (bt.full()) launch();
        }
    if (bt.count) launch();
    if (at != image + data || memcmp(image, want.data(), data) != 0) { printf("batch image differs\n"); return 1; }

    // the general path
    std::vector<ckpt_tile> table(tiles);
    TileBatch tb;
    tb.count = 0;
    uint64_t d = 0, tile = 0;
    for (size_t k = 0; k < ts.size(); k++) {
        const uint32_t j = tb.count++;
        tb.src[j] = uint64_t(ts[k].base + ts[k].lead); tb.data_off[j] = d; tb.nbytes[j] = ts[k].nbytes; tb.first_tile[j] = uint32_t(tile);
        tile += tiles_of(d, ts[k].nbytes, kTileBytes);
        d += (ts[k].nbytes + 4095) / 4096 * 4096;
        tb.first_tile[j + 1] = uint32_t(tile);
        if (tb.count == uint32_t(kTileBatch) || k + 1 == ts.size()) { launch_build_tiles(tb, table.data(), nullptr); tb.count = 0; }
    }
    memset(image, 0x33, data);
    launch_pack(table.data(), tiles, image, 0, nullptr, nullptr, nullptr);
    if (memcmp(image, want.data(), data) != 0) { printf("table image differs\n"); return 1; }
    free(image);
    for (auto &t : ts) free(t.base);
    printf("ok launches %d full_pieces %d full_pages %d\n", launches, full_pieces, full_pages);
    return 0;
}
