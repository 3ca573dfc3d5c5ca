"""Where the kernels find what their loads put into LDS (csrc/d2l.h), compiled for the host: every address that is derived from another one against
the definition of the layout (row r, 16-byte chunk c at r * 128 + 16 * (c ^ swizzle(r))), and the banks that are read together."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2109_04312_amd", "csrc")
SOURCE = """
#include "d2l.h"
using namespace mate;
extern "C" {
int swizzle(int quad, int row) { return quad ? swz_quad(row) : swz(row); }
// first row and chunk of a lane's two loads
void load_lane(int quad, int wave, int lane, int* out) {
  const LoadLane l = quad ? make_load_lane<true>(wave, lane) : make_load_lane<false>(wave, lane);
  out[0] = l.row0; out[1] = l.chunk0;
}
void tile_addresses(unsigned tile, int lane, unsigned* plain /* [4] */, unsigned* trans /* [2 dim blocks][2 halves] */) {
  const OperandLanes o(lane);
  const PlainAddr p(o, tile);
  const TransposedAddr t(o, tile);
  for (int ks = 0; ks < 4; ++ks) plain[ks] = p.a[ks];
  for (int db = 0; db < 2; ++db) { trans[2 * db] = t.lo[db]; trans[2 * db + 1] = t.hi[db]; }
}
// of the 32 rows at `at` in the tiles: [2 halves of a block][2 k] and [4 d][2 halves]
void quad_addresses(unsigned tile, unsigned at, int lane, unsigned* plain, unsigned* trans) {
  const QuadAddr a(QuadLanes(lane), tile);
  for (int h = 0; h < 2; ++h) for (int k = 0; k < 2; ++k) plain[2 * h + k] = a.plain_at(at, h, k);
  for (int d = 0; d < 4; ++d) for (int h = 0; h < 2; ++h) trans[2 * d + h] = a.trans_at(at + h * kHalfBlock, d);
}
}
"""
TILES = [0, 8192, 0x4200, 3 * 8192 + 128]
# lanes of a 16-byte LDS read that are served together
TOGETHER = [np.array([0, 1, 2, 3, 12, 13, 14, 15, 20, 21, 22, 23, 24, 25, 26, 27]), np.array([4, 5, 6, 7, 8, 9, 10, 11, 16, 17, 18, 19, 28, 29, 30, 31])]
TOGETHER += [g + 32 for g in TOGETHER]


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("layout")
    (d / "layout.hip").write_text(SOURCE)
    so = str(d / "layout.so")
    subprocess.run(["hipcc", "--offload-arch=gfx950", "--cuda-host-only", "-O1", "-std=c++17", "-fPIC", "-shared", "-w", f"-I{CSRC}", str(d / "layout.hip"),
                    "-o", so], check=True, capture_output=True)
    return C.CDLL(so)


def place(lib, quad, row, chunk):
    return row * 128 + 16 * (chunk ^ lib.swizzle(quad, row))


def no_bank_twice(addresses):
    """[64] addresses of a 16-byte read: the lanes served together read all of the 64 banks."""
    return all(len(set((addresses[g] // 16) % 16)) == 16 for g in TOGETHER)


@pytest.mark.parametrize("quad", [0, 1])
def test_loads_deposit_by_the_layout(lib, quad):
    out = (C.c_int * 2)()
    for wave in range(4):
        for lane in range(64):
            lib.load_lane(quad, wave, lane, out)
            for i in range(2):   # a load puts lane l's 16 bytes at 16 l of its eight rows
                row, chunk = out[0] + 8 * i, out[1] ^ (2 * i)
                assert place(lib, quad, row, chunk) == (16 * wave + 8 * i) * 128 + 16 * lane


@pytest.mark.parametrize("tile", TILES)
def test_operands_of_32_by_32_tiles(lib, tile):
    plain, trans = (C.c_uint * 4)(), (C.c_uint * 4)()
    seen = np.zeros((4, 64), np.int64)
    for lane in range(64):
        m, hl, i, g = lane & 31, lane >> 5, lane & 15, lane >> 4
        lib.tile_addresses(tile, lane, plain, trans)
        for ks in range(4):
            seen[ks, lane] = plain[ks]
            assert plain[ks] == tile + place(lib, 0, m, 2 * ks + hl)
        for db in range(2):
            for half in range(2):
                row, chunk = 4 * hl + (i >> 2) + 8 * half, 4 * db + 2 * (g & 1) + ((i & 3) >> 1)
                assert trans[2 * db + half] == tile + place(lib, 0, row, chunk) + 8 * (i & 1)
    assert all(no_bank_twice(s) for s in seen)


@pytest.mark.parametrize("at", [0, 32 * 128, 64 * 128, 96 * 128])
@pytest.mark.parametrize("tile", TILES)
def test_operands_of_16_by_16_tiles(lib, tile, at):
    plain, trans = (C.c_uint * 4)(), (C.c_uint * 8)()
    seen = np.zeros((4, 64), np.int64)
    for lane in range(64):
        r, q = lane & 15, lane >> 4
        lib.quad_addresses(tile, at, lane, plain, trans)
        for h in range(2):
            for k in range(2):
                seen[2 * h + k, lane] = plain[2 * h + k]
                assert plain[2 * h + k] == tile + at + place(lib, 1, 8 * (r >> 2) + 4 * h + (r & 3), 4 * k + q)
            for d in range(4):
                assert trans[2 * d + h] == tile + at + place(lib, 1, 8 * q + 4 * h + (r >> 2), 2 * d + ((r & 3) >> 1)) + 8 * (r & 1)
    assert all(no_bank_twice(s) for s in seen)


def test_sixteen_rows_at_four_chunks_read_every_bank(lib):
    for k in range(2):
        assert no_bank_twice(np.array([place(lib, 0, l & 15, 4 * k + (l >> 4)) for l in range(64)]))
