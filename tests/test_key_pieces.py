"""Which bytes of a tile's key rows a lane of the decode kernels fetches, at cache lengths that no test fills: the kernels'
own arithmetic (csrc/skvq_key_pieces.h), compiled for the host, against Python's integers."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
MOST_TOKENS = 2 ** 31 - 65  # SKVQ_MAX_QUANT_TOKENS

SOURCE = """
#include "skvq_key_pieces.h"
extern "C" void key_offsets(int row_bytes, int last_token, int tile, unsigned *out) {
  const unsigned rows = skvq::rows_after_first(last_token, tile);
  for (unsigned x = 0; x < 4; ++x)
    for (unsigned lane = 0; lane < 64; ++lane)
      out[64 * x + lane] = row_bytes == 64 ? skvq::key_piece_offset<64>(lane, x, rows) : skvq::key_piece_offset<32>(lane, x, rows);
}
"""


@pytest.fixture(scope="module")
def offsets(tmp_path_factory):
    d = tmp_path_factory.mktemp("key_pieces")
    (d / "pieces.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-I", os.path.join(ROOT, "paper_2405_06219_amd", "csrc"),
                    str(d / "pieces.cpp"), "-o", str(d / "pieces.so")], check=True)
    fn = C.CDLL(str(d / "pieces.so")).key_offsets
    fn.argtypes = [C.c_int, C.c_int, C.c_int, C.c_void_p]

    def call(row_bytes, last_token, tile):
        out = np.zeros(256, np.uint32)
        fn(row_bytes, last_token, tile, out.ctypes.data)
        return out
    return call


@pytest.mark.parametrize("row_bytes", [32, 64])
@pytest.mark.parametrize("packed", [1, 2, 15, 64, 65, 127] + [2 ** e + d for e in (26, 27, 28, 30) for d in (-63, -1, 0, 1, 6, 64)] +
                         [MOST_TOKENS - 63, MOST_TOKENS])
def test_pieces_are_those_of_the_lanes_tokens(offsets, row_bytes, packed):
    last_tile = (packed - 1) // 64
    for tile in sorted({0, 1, last_tile // 2, last_tile - 2, last_tile - 1, last_tile}):
        if not 0 <= tile <= last_tile:
            continue
        want = []
        for x in range(4):
            for lane in range(64):
                token = 64 * tile + 16 * x + lane % 16
                quarter = lane // 16 if token < packed else 3
                want.append(row_bytes * (min(token, packed - 1) - 64 * tile) + row_bytes // 4 * quarter)
        assert offsets(row_bytes, packed - 1, tile).tolist() == want, tile
