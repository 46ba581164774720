"""The choice of a tile size by tmask_spmm24, compiled from its header and run on the CPU (256 compute units)."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(__file__), "..", "paper_2102_08124_amd", "csrc")
CUS = 256

SOURCE = """
#include "tmask_spmm_choice.hpp"
using namespace tmask;
extern "C" int choose(int64_t rows, int64_t cols, int64_t tokens, int f32) { return spmm_choose(rows, cols, tokens, f32 != 0, %d); }
extern "C" void tile(int v, int64_t *out) { out[0] = kSpmmTile[v].rows; out[1] = kSpmmTile[v].tokens; out[2] = kSpmmTile[v].persistent; }
extern "C" int count() { return kSpmmTiles; }
"""


@pytest.fixture(scope="module")
def choice(tmp_path_factory):
    """(rows, cols, tokens, fp32 results) -> (rows of a tile, tokens of a tile, persistent workgroups per compute unit)"""
    folder = tmp_path_factory.mktemp("choice")
    src, lib = folder / "choice.cpp", folder / "choice.so"
    src.write_text(SOURCE % CUS)
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, "-o", str(lib), str(src)], check=True)
    dll = ctypes.CDLL(str(lib))
    dll.choose.argtypes = [ctypes.c_int64] * 3 + [ctypes.c_int]

    def pick(rows, cols, tokens, f32=False):
        v = dll.choose(rows, cols, tokens, f32)
        assert 0 <= v < dll.count()
        out = (ctypes.c_int64 * 3)()
        dll.tile(v, out)
        return tuple(out)
    return pick


@pytest.mark.parametrize("rows,tokens", [(16, 2 ** 28), (4, 2 ** 28 + 5), (16, 2 ** 31 - 1), (2 ** 28, 16), (2 ** 31 - 4, 1),
                                         (2 ** 20, 2 ** 12), (2 ** 31 - 4, 16384), (2 ** 22, 2 ** 23), (2 ** 15, 2 ** 31 - 128)])
@pytest.mark.parametrize("cols", [64, 1024, 2 ** 22])
def test_every_accepted_product_can_be_launched(choice, rows, cols, tokens):
    """A workgroup of 256 threads per tile reaches the 2^32 work-items of a launch at 2^24 tiles; persistent ones do not."""
    assert -(-rows // 256) * -(-tokens // 128) <= 2 ** 31 - 1        # what the entry point accepts
    tile_rows, tile_tokens, persistent = choice(rows, cols, tokens)
    tiles = -(-rows // tile_rows) * -(-tokens // tile_tokens)
    assert tiles <= 2 ** 31 - 1
    assert (persistent * CUS if persistent else tiles) * 256 < 2 ** 32


# what each tile size took when it was timed (rows, cols, tokens, results: microseconds on 16 x 16, 32 x 32, 64 x 64, 128 x 64,
# 128 x 128, 128 x 256, 256 x 256): thin products, short reductions, and some of the usual ones
TIMED = [
    (16, 64, 1048576, "bf16", [96.9, 168.6, 140.2, 211.6, 36.6, 44.2, 53.0]),
    (1048576, 64, 4, "bf16", [97.0, 161.1, 130.6, 102.5, 30.6, 58.7, 46.5]),
    (64, 1024, 4096, "bf16", [5.4, 3.9, 5.7, 8.0, 9.3, 13.0, 16.6]),
    (4096, 1024, 16, "bf16", [3.2, 3.7, 5.6, 7.8, 8.7, 11.6, 15.7]),
    (1024, 4096, 1003, "bf16", [43.5, 28.5, 15.2, 19.1, 30.4, 40.6, 57.9]),
    (2048, 256, 4096, "bf16", [61.3, 55.7, 26.7, 21.1, 10.0, 10.2, 12.8]),
    (4096, 1024, 1003, "bf16", [44.2, 38.0, 20.9, 16.5, 11.8, 14.2, 19.3]),
    (4096, 1024, 8192, "bf16", [402.5, 347.9, 166.1, 120.8, 63.9, 57.3, 50.7]),
    (256, 64, 262144, "f32", [376.5, 324.3, 167.0, 131.0, 74.2, 63.5, 54.4]),
    (262144, 128, 16, "f32", [30.6, 50.2, 40.7, 31.3, 15.6, 23.8, 21.9]),
    (8, 256, 262144, "f32", [36.6, 58.7, 53.8, 76.8, 23.8, 26.0, 32.0]),
    (1024, 4096, 1003, "f32", [44.0, 28.3, 15.3, 19.4, 32.3, 43.6, 63.0]),
    (1024, 64, 8192, "f32", [43.2, 41.1, 20.2, 17.5, 10.4, 11.2, 14.8]),
    (8192, 64, 8192, "f32", [364.9, 316.1, 138.7, 109.3, 49.6, 53.3, 53.0]),
    (3072, 4096, 3000, "f32", [347.9, 229.6, 118.0, 98.8, 88.4, 89.2, 67.3]),
]


@pytest.mark.parametrize("rows,cols,tokens,out,us", TIMED)
def test_the_choice_is_near_the_fastest_tile(choice, rows, cols, tokens, out, us):
    tiles = [(16, 16), (32, 32), (64, 64), (128, 64), (128, 128), (128, 256), (256, 256)]
    picked = us[tiles.index(choice(rows, cols, tokens, out == "f32")[:2])]
    assert picked <= 1.15 * min(us)        # the fit's largest miss is 13 %


def test_the_products_of_the_gpu_tests_cover_every_tile(choice):
    """Which tile the shapes in test_gpu_spmm.py take: each one with both result types, each that splits the reduction with
    one that takes a wavefront through both of its index buffers and around its ring again and ends within a unit, each
    shared one with whole and partial tiles in one launch, the persistent ones with several tiles to a workgroup."""
    pytest.importorskip("torch")
    from tests import test_gpu_spmm as gpu
    edges = gpu.test_every_tile_size_at_its_edges.pytestmark[0].args[1]
    seen = {}
    for rows, cols, tokens, out in list(edges) + gpu.LONG_AND_THIN:
        tile = choice(rows, cols, tokens, out == "f32")
        seen.setdefault((tile[:2], out), []).append((rows, cols, tokens, tile[2]))
    for size in ((16, 16), (32, 32), (64, 64), (128, 64), (128, 128), (128, 256), (256, 256)):
        for out in ("f32", "bf16"):
            shapes = seen[size, out]
            assert any(r % size[0] and t % size[1] for r, c, t, p in shapes), (size, out)
            tiles = [-(-r // size[0]) * -(-t // size[1]) for r, c, t, p in shapes]
            if shapes[0][3] == 0:
                # a unit is four steps of 64; four wavefronts deal them out, so nine give the first one three
                assert any(c > 8 * 256 for r, c, t, p in shapes), (size, out)
            elif size != (128, 256):                                  # never chosen for more tiles than compute units
                assert max(tiles) > shapes[0][3] * CUS, (size, out)
        if shapes[0][3] == 0:
            assert any(c > 8 * 256 and c % 256 for o in ("f32", "bf16") for r, c, t, p in seen[size, o]), size
