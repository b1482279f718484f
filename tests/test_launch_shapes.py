"""CPU-only checks of the launch shapes (csrc/grid.hpp, compiled for the host):
every block of a call is launched, within what a launch may hold."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2607_27090_amd", "csrc")
SOURCE = r"""
#include "grid.hpp"
extern "C" void fold(int64_t blocks, int threads, uint32_t* xy) {
    const is::GridXY g = is::fold_grid(blocks, threads);
    xy[0] = g.x;
    xy[1] = g.y;
}
extern "C" int64_t shares(int64_t rows, int qtiles, int cus, int* blocks) {
    const is::RowShares g = is::row_shares(rows, 256, 32, qtiles, cus);
    *blocks = g.blocks;
    return g.rows;
}
extern "C" void token_rule(int64_t max_tokens, int64_t parts, int target, is::TokenRule* r) {
    *r = is::token_rule(max_tokens, parts, target, 32);
}
extern "C" void token_share(int m, unsigned block, const is::TokenRule* r, int* fl) {
    const is::TokenShare s = is::token_share(m, block, *r);
    fl[0] = s.first;
    fl[1] = s.last;
}
extern "C" int pieces(int nq, int k, int max_tokens, int64_t row_elements, int cus) {
    return is::inject_pieces(nq, k, max_tokens, row_elements, cus);
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("shapes")
    src, so = d / "shapes.cpp", d / "shapes.so"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC,
                    str(src), "-o", str(so)], check=True)
    return ctypes.CDLL(str(so))


def _fold(lib, blocks, threads):
    xy = (ctypes.c_uint32 * 2)()
    lib.fold(ctypes.c_int64(blocks), threads, xy)
    return xy[0], xy[1]


@pytest.mark.parametrize("threads", [256, 512])
@pytest.mark.parametrize("blocks", [1, 8, 255, 2 ** 22, 2 ** 23 - 1, 2 ** 23, 2 ** 24 - 1, 2 ** 24,
                                    2 ** 24 + 8, 2 ** 26 + 1, 35_000_000, 2 ** 31])
def test_folded_grids_hold_every_block(lib, blocks, threads):
    # (2^31 rows in tiles of 32 are 2^26 blocks; 2^24 blocks of 256 threads are
    # one thread more than a dimension of a launch takes)
    x, y = _fold(lib, blocks, threads)
    assert x * threads < 2 ** 32 and 1 <= y <= 65535
    assert x * (y - 1) < blocks <= x * y
    if blocks * threads < 2 ** 32:
        assert (x, y) == (blocks, 1)
    else:
        assert x % 8 == 0


def test_blocks_past_a_grid_are_refused(lib):
    assert _fold(lib, 2 ** 41, 256) == (0, 0)


@pytest.mark.parametrize("rows", [1, 255, 256, 500, 3000, 16_384, 45_925, 100_000, 934_464])
def test_row_shares_keep_the_cus_busy(lib, rows):
    lib.shares.restype = ctypes.c_int64
    cus, tiles = 256, -(-rows // 256)
    for qtiles in [1, 2, 3, 4, 5, 7, 16, 65, 100, 127, 128, 129, 160, 170, 200, 255, 256]:
        b = ctypes.c_int()
        share = lib.shares(ctypes.c_int64(rows), qtiles, cus, ctypes.byref(b))
        blocks = b.value
        assert share % 32 == 0 and 1 <= blocks <= min(cus, tiles) and blocks * share >= rows
        if qtiles == 1:
            assert blocks == min(cus, tiles)
        # row tiles one CU after the other has to take, against an even split of
        # all tiles over all CUs (a block takes whole tiles: at most one more)
        walk = -(-blocks * qtiles // cus) * -(-share // 256)
        even = tiles * qtiles / cus
        assert walk <= 1.34 * even + 1, (qtiles, blocks, share, walk, even)


@pytest.mark.parametrize("capacity", [1, 16, 17, 300, 640, 2560, 16_500, 131_072, 2 ** 31 - 1])
@pytest.mark.parametrize("parts", [1, 2, 4, 64, 845, 1000, 65_535])
def test_token_shares_follow_what_is_placed(lib, capacity, parts):
    target, i64 = 1024, ctypes.c_int64
    rule = (ctypes.c_uint32 * 6)()
    lib.token_rule(i64(capacity), i64(parts), target, rule)
    blocks, most = rule[0], rule[3]
    # no more than four times `target` blocks, or one per part
    assert 1 <= blocks <= -(-capacity // 16) and blocks * parts <= max(4 * target, parts)
    # 512 tokens a block where the blocks hold the capacity in such shares
    assert most == (32 if blocks * 512 >= capacity else 2 ** 32 - 1)
    for m in {0, 1, 15, 16, 17, 33, 300, 2500, capacity // 2, capacity}:
        if m > capacity or blocks > 5000:
            continue
        at, longest = 0, 0
        fl = (ctypes.c_int * 2)()
        for b in range(blocks):
            lib.token_share(m, b, rule, fl)
            if fl[0] < fl[1]:
                assert fl[0] == at and fl[0] % 16 == 0
                at, longest = fl[1], max(longest, fl[1] - fl[0])
        assert at == max(m, 0) and longest <= 16 * most
        # every CU's share of what is placed, whatever the capacity
        groups = -(-m // 16)
        if m < capacity // 2:
            assert longest <= 16 * max(1, -(-groups // blocks), parts * groups // target) + 16 * (m > 2 ** 25)
        else:
            assert longest <= 16 * max(1, parts * -(-capacity // 16) // target)


@pytest.mark.parametrize("nq,k,row_elements,want", [
    (1, 50, 32 * 1024, 1), (7, 100, 80 * 1024, 1), (8, 3, 32 * 1024, 1), (64, 10, 32 * 1024, 4),
    (64, 3, 32 * 1024, 2), (65_535, 1024, 80 * 1024, 4)])
def test_injection_workgroups_do_not_follow_the_capacity(lib, nq, k, row_elements, want):
    # a buffer for longer requests than are placed costs no workgroups
    for capacity in (64 * k, 8192 + 64 * k, 2 ** 31 - 1):
        assert lib.pieces(nq, k, capacity, ctypes.c_int64(row_elements), 256) == want
    assert lib.pieces(nq, k, 0, ctypes.c_int64(row_elements), 256) == 1
