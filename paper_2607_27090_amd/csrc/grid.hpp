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

}  // namespace is
