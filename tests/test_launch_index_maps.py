"""Host-side walk (no GPU) of the index functions the kernels share with it: every work item of a launch is taken exactly
once, whatever stands in front of it in the grid."""
import ctypes
import os
import shutil
import subprocess

import pytest

from paper_2509_16495_amd import build as BLD

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++ to compile the index functions for the host")

SOURCE = r"""
#include "tile_order.h"
#include "token_rows.h"
#include <vector>
using namespace shiftattn;
// work items (tile rank, key range, (sequence, head)) of a grid that are out of range or not taken exactly once
extern "C" int items_missed(int decode_wgs, int n_sh, int ranks, int n_splits, int range_major, int rotate) {
    const int items = n_sh * ranks * n_splits;
    std::vector<int> taken(items, 0);
    int bad = 0;
    for (int block = decode_wgs; block < decode_wgs + items; ++block) {
        const TileItem t = tile_item(block, decode_wgs, n_sh, ranks, n_splits, range_major != 0, rotate != 0);
        if (t.rank < 0 || t.rank >= ranks || t.split < 0 || t.split >= n_splits || t.sh < 0 || t.sh >= n_sh) ++bad;
        else ++taken[(t.rank * n_splits + t.split) * n_sh + t.sh];
    }
    for (const int n : taken) bad += n != 1;
    return bad;
}
// (sequence, head) of one workgroup
extern "C" int sh_of(int block, int decode_wgs, int n_sh, int ranks, int n_splits, int range_major, int rotate) {
    return tile_item(block, decode_wgs, n_sh, ranks, n_splits, range_major != 0, rotate != 0).sh;
}
// rows of the token tiles of a result of M_out rows, M of which are tokens, whose load would leave the M rows, go backwards
// from the tile's origin, or fetch another token than the row's own (the last one for padding rows)
extern "C" int rows_wrong(int M, int M_out, int tile) {
    int bad = 0;
    for (int m0 = 0; m0 < M_out; m0 += tile)
        for (int row = 0; row < tile; ++row) {
            const int from = tile_origin(m0, M), behind = tile_row(m0, row, M), token = from + behind;
            bad += behind < 0 || from < 0 || token >= M || token != (m0 + row < M ? m0 + row : M - 1);
        }
    return bad;
}
"""


@pytest.fixture(scope="module")
def maps(tmp_path_factory):
    d = tmp_path_factory.mktemp("maps")
    src, lib = os.path.join(str(d), "maps.cpp"), os.path.join(str(d), "maps.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.check_call(["g++", "-std=c++20", "-O1", "-shared", "-fPIC", "-I", BLD.CSRC, src, "-o", lib])
    return ctypes.CDLL(lib)


@pytest.mark.parametrize("n_sh", [1, 2, 3, 4, 5, 6, 7, 8, 12, 16, 20, 24, 28, 40, 44, 48, 100])
def test_prefill_grids_take_every_work_item_once(maps, n_sh):
    """With and without decode workgroups in front: counts that divide the runs of n_sh workgroups and counts that do not
    (the planner hands out what the tiles leave of 256, or 32 to 192)."""
    for decode_wgs in (0, 8, 32, 64, 96, 128, 192, 196, 201, 255):
        for ranks in (1, 2, 3, 8, 57):
            for n_splits in (1, 2, 3, 16):
                for range_major in (0, 1):
                    for rotate in (0, 1):
                        args = (decode_wgs, n_sh, ranks, n_splits, range_major, rotate)
                        assert maps.items_missed(*args) == 0, args


@pytest.mark.parametrize("n_sh", [4, 8, 12, 24])
def test_rotation_shows_every_die_all_sequences(maps, n_sh):
    """Workgroup i runs on die i % 8: with a rotation a die meets every (sequence, head) within a few rounds."""
    for decode_wgs in (0, 96, 196):
        for die in range(8):
            blocks = [b for b in range(decode_wgs, decode_wgs + n_sh * 64) if b % 8 == die]
            assert {maps.sh_of(b, decode_wgs, n_sh, 64, 1, 0, 1) for b in blocks} == set(range(n_sh))


@pytest.mark.parametrize("tile", [128, 256])
def test_projection_tiles_load_rows_that_exist(maps, tile):
    """Tiles that end in padding rows and tiles of padding rows only, whose origin lies past the last token."""
    for M in (1, 2, 127, 128, 129, 255, 256, 257, 384, 512, 701):
        for M_out in (M, M + 1, M + 7, M + tile - 1, M + tile, M + tile + 1, M + 3 * tile):
            assert maps.rows_wrong(M, M_out, tile) == 0, (M, M_out)


@pytest.mark.parametrize("n_sh", [4, 8])
def test_rotation_shows_every_engine_all_sequences(maps, n_sh):
    """Workgroup i runs on die i % 8, shader engine (i / 8) % 4 of it: with a rotation of few (sequence, head) each of the 32 meets every (sequence, head)
    about equally often, whatever decode workgroups stand in front and in either order of the grid."""
    for decode_wgs in (0, 67, 96):
        for ranks, n_splits, range_major in ((32 * n_sh, 1, 0), (8 * n_sh, 4, 0), (8 * n_sh, 4, 1)):
            seen = [[0] * n_sh for _ in range(32)]
            for b in range(decode_wgs, decode_wgs + n_sh * 32 * n_sh):
                seen[b % 32][maps.sh_of(b, decode_wgs, n_sh, ranks, n_splits, range_major, 1)] += 1
            assert min(min(x) for x in seen) >= 0.6 * n_sh and max(max(x) for x in seen) <= 1.6 * n_sh, (decode_wgs, ranks, n_splits)


@pytest.mark.parametrize("n_sh", [12, 16, 20, 24])
def test_rotation_of_many_goes_on_by_one_a_run(maps, n_sh):
    """Every engine shown all of them costs more than it gives from 12 on."""
    runs = [[maps.sh_of(r * n_sh + i, 0, n_sh, 64, 1, 0, 1) for i in range(n_sh)] for r in range(64)]
    assert runs == [[(i - r) % n_sh for i in range(n_sh)] for r in range(64)]
