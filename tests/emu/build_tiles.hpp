// The tile table of a tensor list, built batch by batch from (source, offset, size) alone: the second, independent construction
// that the planner's table and the pack kernels are compared with. Tile i of a tensor whose padded extent is [d0, dend) of the data
// region: the extent is cut at its start and at every multiple of the tile size.
#pragma once
#include "../../paper_2406_10707_amd/csrc/plan.hpp"

namespace dsllm {

constexpr int kTileBatch = 96;

struct TileBatch {
    uint64_t src[kTileBatch];          // address of the tensor's first byte
    uint64_t data_off[kTileBatch];     // offset of the tensor in the data region (a multiple of 4096)
    uint64_t nbytes[kTileBatch];
    uint32_t first_tile[kTileBatch + 1];   // index of the tensor's first tile in the table; [count] = one past the batch's last
    uint32_t count;
};

inline void launch_build_tiles(const TileBatch &bt, ckpt_tile *table, void *) {
    const uint64_t T = kTileBytes;
    for (uint32_t k = 0; k < bt.count; k++) {
        const uint64_t d0 = bt.data_off[k], dend = d0 + (bt.nbytes[k] + 4095) / 4096 * 4096;
        for (uint32_t i = 0; i < bt.first_tile[k + 1] - bt.first_tile[k]; i++) {
            const uint64_t start = i == 0 ? d0 : (d0 / T + i) * T, cut = (d0 / T + i + 1) * T, stop = cut < dend ? cut : dend;
            const uint64_t left = start - d0 >= bt.nbytes[k] ? 0 : bt.nbytes[k] - (start - d0);
            ckpt_tile t{};
            t.src = bt.src[k] + (start - d0);
            t.dst_off = start;
            t.copy_bytes = uint32_t(left < stop - start ? left : stop - start);
            t.total_bytes = uint32_t(stop - start);
            table[bt.first_tile[k] + i] = t;
        }
    }
}

}  // namespace dsllm
