// Launch shapes: host arithmetic, and what the kernels share of it.
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

// Paged logits: a launch has TokenRule::blocks blocks per request and head share
// (`parts` of those), about `target` in all at full capacity, so that a large
// max_tokens costs no blocks. The blocks of a request share out its m placed
// tokens, in groups of 16: as many groups each as give `target` blocks if every
// request placed m, or, with m close to the capacity, max_tokens. (With shares by
// capacity, 300 tokens of 131,072 were one block's work: 32 requests of 32 heads
// of 32 140 us, by m 14.) The kernel is small, and its first loads wait for its
// share: with divisions a call took 0.3 us longer, so the launch brings
// reciprocals.
struct TokenRule {
    uint32_t blocks;
    uint32_t per_block;  // 2^32 / blocks, rounded up
    uint32_t per_m;      // groups of a block for each of a request's, in 65536ths
    uint32_t most;       // groups of a block at most
    uint32_t half, full; // from `half` groups on, half of the capacity: `full` a block
};
struct TokenShare {
    int32_t first, last;  // tokens [first, last)
};

constexpr int64_t token_groups(int64_t tokens) { return (tokens + 15) / 16; }

// `most`: groups a block should have at most; kept while that takes no more than
// four times `target` blocks (past it the empty ones of a short request cost
// more than they give: the hardware starts one every few ns).
inline TokenRule token_rule(int64_t max_tokens, int64_t parts, int target, uint32_t most) {
    const int64_t groups = token_groups(max_tokens);
    int64_t per = parts * groups / target > 1 ? parts * groups / target : 1;
    if (per > most && (groups + most - 1) / most * parts <= 4 * (int64_t)target) per = most;
    const int64_t blocks = (groups + per - 1) / per;
    const int64_t per_m = blocks > 1 && parts < target ? parts * 65536 / target : 65536;
    return {(uint32_t)blocks, blocks > 1 ? (uint32_t)((((uint64_t)1 << 32) + blocks - 1) / blocks) : 0,
            (uint32_t)per_m, groups <= blocks * most ? most : UINT32_MAX,
            (uint32_t)((groups + 1) / 2), (uint32_t)per};
}

constexpr TokenShare token_share(int32_t m, uint32_t block, const TokenRule& rule) {
    const uint32_t groups = m > 0 ? ((uint32_t)m + 15) / 16 : 0;
    // groups over blocks, rounded up (by one too many past 2^32 / blocks groups)
    const uint32_t even = (uint32_t)(((uint64_t)(groups + rule.blocks - 1) * rule.per_block) >> 32);
    uint32_t per = (uint32_t)(((uint64_t)groups * rule.per_m) >> 16);
    per = per < even ? even : per;
    per = per > rule.most ? rule.most : per;
    per = groups >= rule.half ? rule.full : per;
    const uint64_t first = (uint64_t)block * per;
    if ((uint32_t)(first >> 32) != 0 || (uint32_t)first >= groups) return {0, 0};
    const uint32_t f = (uint32_t)first;
    return {(int32_t)(f * 16), f + per >= groups ? m : (int32_t)((f + per) * 16)};
}

// Workgroups per CU of an injection. The tokens a request places differ (ten
// facts of 16 to 64 tokens: 280 to 510), so with many requests equal shares of
// the CUs end far apart: from 8 requests on, a request's share is cut into
// several workgroups that the hardware hands out as CUs come free. One more per
// CU costs 4 to 5 us whatever it finds to do (the hardware starts a workgroup
// of 12 waves every 20 ns), so there is one for each 4 MiB of a CU's expected
// bytes. What will be placed is not known here: max_tokens is a buffer's size
// (8 requests of 50 tokens in buffers for 32,768 took 94 us instead of 25 with
// workgroups by max_tokens) and facts are a few dozen tokens, so 32 per fact are
// expected. Workgroups per CU 1 / 2 / 4 / 8 / 16, us: 64 requests of 10 facts of
// 16 to 64 tokens 1,518 / 1,452 / 1,417 / 1,418 / 1,389, of 3 facts 454 / 413 /
// 395 / 393 / 402; 16 of 20 facts 649 / 654 / 655 / 659 / 672; 64 of 10 facts of
// 4 to 12 tokens 269 / 270 / 271 / 277 / 294, of one or two tokens 57 / 61 / 69 /
// 81 / 117; but 4 requests of 50 facts 413 / 426 / - / 445 / 491.
inline int inject_pieces(int nq, int k, int max_tokens, int64_t row_elements, int cus) {
    if (nq < 8) return 1;
    const int64_t expected = (int64_t)k * 32 < max_tokens ? (int64_t)k * 32 : max_tokens;
    const double bytes = 8.0 * nq * (double)expected * (double)row_elements;  // K and V, in and out
    const double pieces = 1.0 + bytes / ((double)(4 << 20) * cus);
    return pieces < 4.0 ? (int)pieces : 4;
}

}  // namespace is
