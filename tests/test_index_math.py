"""Index arithmetic of the kernels that plain C++ can run: headers of csrc that
hold nothing else are compiled with the host compiler and checked by counting."""
import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include "sj_tiles.h"
// Tiles of workgroup b of `grid`, as pt << 32 | qt; returns their number.
template <bool TRI>
static uint32_t walk(uint32_t n_pt, uint32_t n_qt, uint32_t b, uint32_t grid, uint64_t *out)
{
    sjk::TileWalk<TRI> w(n_pt, n_qt, b, grid);
    sjk::TileAt t;
    uint32_t n = 0;
    while (w.next(t))
        out[n++] = (uint64_t)t.pt << 32 | t.qt;
    return n;
}
extern "C" uint32_t tiles(int tri, uint32_t n_pt, uint32_t n_qt, uint32_t b, uint32_t grid,
                          uint64_t *out)
{
    return tri ? walk<true>(n_pt, n_qt, b, grid, out) : walk<false>(n_pt, n_qt, b, grid, out);
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    d = tmp_path_factory.mktemp("index_math")
    (d / "index_math.cpp").write_text(SOURCE)
    so = str(d / "index_math.so")
    subprocess.run([cxx, "-std=c++17", "-O1", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2006_12608_amd", "csrc"), str(d / "index_math.cpp"),
                    "-o", so], check=True)
    return ctypes.CDLL(so)


def workgroup_tiles(lib, tri, n_pt, n_qt, grid):
    buf = (ctypes.c_uint64 * (n_pt * n_qt + 1))()
    out = []
    for b in range(grid):
        n = lib.tiles(int(tri), n_pt, n_qt, b, grid, buf)
        out.append([(v >> 32, v & 0xffffffff) for v in buf[:n]])
    return out


def check(per_wg, want):
    flat = [t for wg in per_wg for t in wg]
    assert len(flat) == len(set(flat)) == len(want) and set(flat) == want
    # dealt evenly: no workgroup takes two tiles more than another
    assert max(map(len, per_wg)) - min(map(len, per_wg)) <= 1


@pytest.mark.parametrize("n_pt,n_qt", [(1, 1), (1, 40), (40, 1), (7, 9), (8, 8), (9, 17), (16, 33),
                                       (33, 16), (18, 19), (64, 64), (65, 71)])
def test_streamed_tiles(lib, n_pt, n_qt):
    want = {(p, q) for p in range(n_pt) for q in range(n_qt)}
    for grid in (1, min(256, n_pt * n_qt), min(304, n_pt * n_qt)):
        check(workgroup_tiles(lib, False, n_pt, n_qt, grid), want)


@pytest.mark.parametrize("n", [1, 2, 7, 8, 9, 15, 16, 17, 31, 32, 33, 64, 65, 96, 128, 200])
def test_streamed_triangle_tiles(lib, n):
    """A self-join's tiles: those on and above the diagonal, each once, and every
    workgroup its even share (8192, 16384, 24576 and 32768 rows among them)."""
    want = {(p, q) for p in range(n) for q in range(p, n)}
    for grid in (1, min(256, len(want)), min(304, len(want))):
        check(workgroup_tiles(lib, True, n, n, grid), want)
