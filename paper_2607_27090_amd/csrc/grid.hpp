// Launch shapes: host arithmetic only.
#pragma once

#include <stdint.h>

namespace is {

struct GridXY {
    uint32_t x, y;  // x == 0: the blocks do not fit a grid
};

// `blocks` (at least 1) blocks of `threads` threads as a grid of x * y >= blocks
// in the order y * x + x: a dimension of a launch must hold fewer than 2^32
// threads (2^24 blocks of 256), and y at most 65,535 blocks. A folded x is a
// multiple of 8, so block b still goes to XCD b % 8.
inline GridXY fold_grid(int64_t blocks, int threads) {
    const int64_t most = (((int64_t)1 << 32) - 1) / threads;
    if (blocks <= most) return {(uint32_t)blocks, 1};
    const int64_t x = most / 8 * 8;
    const int64_t y = (blocks + x - 1) / x;
    return y <= 65535 ? GridXY{(uint32_t)x, (uint32_t)y} : GridXY{0, 0};
}

struct RowShares {
    int blocks;    // per query tile, at most `cus`
    int64_t rows;  // rows of one, a multiple of `step`
};

// Shares of `rows` rows, walked in tiles of `tile`, for each of `qtiles` query
// tiles, one block per CU at a time. One round of blocks over all query tiles,
// so that a block walks several row tiles and its loads run on across them
// (1,024 queries over 45,925 rows, d = 768: 64 x 4 blocks of three tiles 94 us,
// 180 x 4 of one 111); more rounds of smaller shares where one leaves too many
// CUs without a block (129 query tiles: 129 of 256). A round costs its largest
// share's tiles and about a quarter of one to start.
inline RowShares row_shares(int64_t rows, int tile, int step, int qtiles, int cus) {
    const int64_t tiles = (rows + tile - 1) / tile;
    RowShares best{1, 0};
    double least = 0;
    for (int round = 1; round <= 8; ++round) {
        int64_t g = (int64_t)round * cus / qtiles;
        if (g < 1) g = 1;
        if (g > cus) g = cus;
        if (g > tiles) g = tiles;
        if (g < 1) g = 1;
        int64_t share = (rows + g - 1) / g;
        share = (share + step - 1) / step * step;
        const int64_t rounds = (g * qtiles + cus - 1) / cus;
        const double cost = (double)rounds * ((double)((share + tile - 1) / tile) + 0.25);
        if (best.rows == 0 || cost < least) {
            best = {(int)g, share};
            least = cost;
        }
        if (qtiles == 1) break;
    }
    return best;
}

}  // namespace is
