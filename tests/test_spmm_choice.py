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
extern "C" int choose(int64_t rows, int64_t cols, int64_t tokens) { return spmm_choose(rows, cols, tokens, %d); }
extern "C" void tile(int v, int64_t *out) { out[0] = kSpmmTile[v].rows; out[1] = kSpmmTile[v].tokens; out[2] = kSpmmTile[v].persistent; }
extern "C" int count() { return kSpmmTiles; }
"""


@pytest.fixture(scope="module")
def choice(tmp_path_factory):
    """(rows, cols, tokens) -> (rows of a tile, tokens of a tile, persistent workgroups per compute unit)"""
    folder = tmp_path_factory.mktemp("choice")
    src, lib = folder / "choice.cpp", folder / "choice.so"
    src.write_text(SOURCE % CUS)
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, "-o", str(lib), str(src)], check=True)
    dll = ctypes.CDLL(str(lib))
    dll.choose.argtypes = [ctypes.c_int64] * 3

    def pick(rows, cols, tokens):
        v = dll.choose(rows, cols, tokens)
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
