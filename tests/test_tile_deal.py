"""Which tile a workgroup of a product computes (csrc/tile_deal.h, csrc/division.h), compiled for the host."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2109_04312_amd", "csrc")
SOURCE = """
#include "tile_deal.h"
using namespace mate;
extern "C" {
void divide(long n, const int* x, const int* d, int* k, int* rest) {
  for (long i = 0; i < n; ++i) k[i] = uniform_div_any(x[i], d[i], rest[i]);
}
// (sequence, place in it, feature tile) of every workgroup of grid rows [y0, y1), -1 where it has none; returns the rows there are
int deal(int tokens, int features, int rows, int by_feature, int tiles_each, int y0, int y1, int* out) {
  const TileDeal d = {tokens, features, rows, by_feature};
  for (int y = y0; y < y1 && y < d.grid_y(); ++y)
    for (int x = 0; x < d.grid_x(); ++x, out += 3) {
      int token_tile;
      if (dealt_tile(d, x, y, token_tile, out[2])) out[0] = sequence_of(token_tile, tiles_each, out[1]);
      else out[0] = out[1] = out[2] = -1;
    }
  return d.grid_y();
}
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("deal")
    (d / "deal.cpp").write_text(SOURCE)
    so = str(d / "deal.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-I/opt/rocm/include", f"-I{CSRC}",
                    str(d / "deal.cpp"), "-o", so], check=True)
    return C.CDLL(so)


def _deal(lib, tokens, features, by_feature, tiles_each, y0=0, y1=1 << 30):
    major, minor = (features, tokens) if by_feature else (tokens, features)
    rows = major // 8
    y1 = min(y1, rows + 1)
    out = np.full(((y1 - y0) * 8 * minor, 3), -1, np.int32)
    n = lib.deal(tokens, features, rows, int(by_feature), tiles_each, y0, y1, out.ctypes.data_as(C.c_void_p))
    assert n == (major + 7) // 8
    return out[out[:, 0] >= 0].astype(np.int64)


@pytest.mark.parametrize("by_feature", [False, True])
@pytest.mark.parametrize("B,tiles_each,features", [(1, 1, 1), (1, 7, 12), (1, 8, 3), (3, 3, 5), (5, 5, 9), (13, 1, 2), (43, 17, 12), (3001, 1, 2)])
def test_every_tile_is_dealt_once(lib, B, tiles_each, features, by_feature):
    got = _deal(lib, B * tiles_each, features, by_feature, tiles_each)
    want = np.stack(np.meshgrid(np.arange(B), np.arange(tiles_each), np.arange(features), indexing="ij"), -1).reshape(-1, 3)
    assert np.array_equal(got[np.lexsort(got.T[::-1])], want)


@pytest.mark.parametrize("tiles_each", [1, 3])
@pytest.mark.parametrize("at", [1 << 21, 1 << 24, 1 << 25, 1 << 26, (1 << 28) - 64])
def test_token_tiles_of_very_many_sequences(lib, at, tiles_each):
    """The sequence is a quotient as large as the number of sequences: it is exact, whatever that is."""
    tokens = (at + 43) // tiles_each * tiles_each
    y0 = at // 8 - 4
    got = _deal(lib, tokens, 2, False, tiles_each, y0)
    tile = np.repeat(np.arange(8 * y0, tokens), 2)
    got = got[np.lexsort(got.T[::-1])]
    assert np.array_equal(got[:, 0], tile // tiles_each) and np.array_equal(got[:, 1], tile % tiles_each)


def test_division(lib):
    rng = np.random.default_rng(0)
    d = np.concatenate([np.arange(1, 300), 2 ** np.arange(9, 30), rng.integers(300, 1 << 30, 200)])
    near = np.concatenate([[0, 1], *(2 ** e + np.arange(-3, 4) for e in (20, 21, 22, 24, 25, 26, 30)), [2 ** 31 - 1]])
    x, d = (v.reshape(-1) for v in np.meshgrid(np.concatenate([near, rng.integers(0, 2 ** 31, 300)]), d))
    near = (x // d) * d   # beside a change of the quotient
    x, d = np.concatenate([x, near, np.maximum(near - 1, 0)]).astype(np.int32), np.concatenate([d, d, d]).astype(np.int32)
    k, rest = np.empty_like(x), np.empty_like(x)
    p = lambda a: a.ctypes.data_as(C.c_void_p)
    lib.divide(C.c_long(len(x)), p(x), p(d), p(k), p(rest))
    assert np.array_equal(k, x // d) and np.array_equal(rest, x % d)
