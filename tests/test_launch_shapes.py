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
