"""How the tiles of a level are dealt to the XCDs (no GPU): the header that says so, compiled for the host."""
import ctypes
import subprocess

import numpy as np
import pytest

from paper_2507_04123_amd import build as hip_build

_SHIM = """#include "xcd_tiles.h"
template <int RUN> static void deal(int64_t n, int64_t* count, int64_t* tile) {   // tile[n]: the XCDs' tiles one after the other
  for (uint32_t x = 0; x < 8; ++x) {
    count[x] = emc2_xcd_tiles<RUN>(x, n);
    for (int64_t s = 0; s < count[x]; ++s) *tile++ = emc2_xcd_tile<RUN>(x, s, n);
  }
}
extern "C" void deal_to(int run, int64_t n, int64_t* count, int64_t* tile) {
  if (run == 4) deal<4>(n, count, tile); else if (run == 16) deal<16>(n, count, tile); else deal<32>(n, count, tile);
}
"""


@pytest.fixture(scope="module")
def deal(tmp_path_factory):
    d = tmp_path_factory.mktemp("xcd_tiles")
    (d / "shim.cpp").write_text(_SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-shared", "-fPIC", "-I", hip_build.CSRC,
                    str(d / "shim.cpp"), "-o", str(d / "shim.so")], check=True)
    f = ctypes.CDLL(str(d / "shim.so")).deal_to
    f.argtypes = [ctypes.c_int, ctypes.c_int64, ctypes.c_void_p, ctypes.c_void_p]

    def run(length, n):
        count, tile = np.zeros(8, np.int64), np.full(n + 8 * length + 8, -1, np.int64)
        f(length, n, count.ctypes.data, tile.ctypes.data)
        return count, tile
    return run


@pytest.mark.parametrize("run", [4, 16, 32])
def test_every_tile_once_and_even_shares(deal, run):
    """Whatever the number of tiles: each is dealt once, and no XCD has more than one above another.  A launch's grid is sized by
    an eighth of the capacity's tiles, rounded up."""
    for n in list(range(0, 3 * 8 * run + 9)) + [12345, 65536 - 1, 66000 // 32, (1 << 26) // 32 + 5, 1 << 20]:
        count, tile = deal(run, n)
        assert count.sum() == n and count.max() <= -(-n // 8) and count.min() >= n // 8, n
        assert np.array_equal(np.sort(tile[:n]), np.arange(n)) and (tile[n:] == -1).all(), n


@pytest.mark.parametrize("run", [4, 16, 32])
def test_runs_in_turn(deal, run):
    """Whole turns: runs of `run` neighbouring tiles, one XCD after the other."""
    n = 5 * 8 * run
    count, tile = deal(run, n)
    assert (count == 5 * run).all()
    t = np.arange(n).reshape(5, 8, run).transpose(1, 0, 2).reshape(-1)
    assert np.array_equal(tile[:n], t)
