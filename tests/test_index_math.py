"""Index arithmetic of the kernels that plain C++ can run: headers of csrc that
hold nothing else are compiled with the host compiler and checked by counting."""
import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include "sj_lsh_layout.h"
#include "sj_search.h"
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
// Keys: 5 in [first, end), 9 from there on.
extern "C" uint32_t run_end_of(uint32_t first, uint32_t end, uint32_t p, uint32_t n)
{
    return sjl::run_end([=](uint32_t i) { return i < first ? 1ull : i < end ? 5ull : 9ull; }, p, n, 5);
}
extern "C" uint32_t entries(uint32_t blk, uint32_t tile, uint32_t n)
{
    return sjl::block_entries(blk, tile, n);
}
extern "C" void layout(const uint64_t *n, uint64_t *out)
{
    sjl::ScratchNeeds c = {};
    c.n_p = n[0], c.n_q = n[1], c.L = n[2], c.self = n[3], c.copy_row = n[4], c.norm = n[5];
    c.fingerprint = n[6], c.hash_ws = n[7], c.widened = n[8], c.sort_ws = n[9];
    c.find_blocks = n[10], c.records = n[11], c.chunks = n[12], c.scan_partials = n[13];
    c.own_pairs = n[14], c.held_bytes = n[15], c.workgroups = n[16];
    const sjl::ScratchLayout y = sjl::scratch_layout(c);
    const size_t v[] = {y.row_p, y.row_q, y.norm_p, y.norm_q, y.key_p, y.key_q, y.perm_p, y.perm_q,
                        y.counters, y.partials, y.hash_ws, y.widened, y.sorted_p, y.sorted_q,
                        y.sort_ws, y.found, y.n_found, y.found_off, y.rec_t, y.rec_pq, y.n_desc,
                        y.n_tile, y.desc_off, y.tile_off, y.list_p, y.list_q, y.tag_p, y.tag_q,
                        y.desc_info, y.desc_pq, y.fp_p, y.fp_q, y.own, y.n_held, y.next, y.held,
                        y.held_bytes, y.total};
    for (unsigned i = 0; i < sizeof v / sizeof *v; ++i)
        out[i] = v[i];
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
    lib = ctypes.CDLL(so)
    lib.run_end_of.restype = lib.entries.restype = ctypes.c_uint32
    return lib


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


NAMES = ("row_p row_q norm_p norm_q key_p key_q perm_p perm_q counters partials hash_ws widened "
         "sorted_p sorted_q sort_ws found n_found found_off rec_t rec_pq n_desc n_tile desc_off "
         "tile_off list_p list_q tag_p tag_q desc_info desc_pq fp_p fp_q own n_held next held held_bytes "
         "total").split()
# the steps of a call (0 hash, 1 sorts, 2 bucket search, 3 records, 4 fingerprints
# and packing, 5 join) from an array's first write to its last read
LIVE = {"hash_ws": (0, 0), "widened": (0, 0), "perm_p": (1, 5), "perm_q": (1, 5),
        "sorted_p": (1, 2), "sorted_q": (1, 2), "sort_ws": (1, 2), "found": (2, 3),
        "n_found": (2, 3), "found_off": (2, 3), "rec_t": (3, 4), "rec_pq": (3, 4), "n_desc": (4, 4),
        "n_tile": (4, 4), "desc_off": (4, 4), "tile_off": (4, 4), "list_p": (4, 5),
        "list_q": (4, 5), "tag_p": (4, 5), "tag_q": (4, 5), "desc_info": (4, 5), "desc_pq": (4, 5),
        "fp_p": (4, 5), "fp_q": (4, 5), "own": (5, 5), "n_held": (5, 5), "next": (5, 5),
        "held": (5, 5)}


@pytest.mark.parametrize("n_p,n_q", [(1, 1), (700, 300), (50000, 50000), (1 << 20, 1 << 20),
                                     (1000, 1 << 24), (1 << 24, 1000), (3 << 20, 5 << 20)])
@pytest.mark.parametrize("L", [1, 2, 16, 64, 200])
@pytest.mark.parametrize("self_join", [False, True])
@pytest.mark.parametrize("long_rows", [False, True])
def test_lsh_scratch_layout(lib, n_p, n_q, L, self_join, long_rows):
    """Arrays that are needed at the same time never overlap, and without the room for
    its own output and held records a call needs no more than the arrays one after the other took when
    none shared its place (so no call that fitted the card stops fitting)."""
    if self_join:
        n_q = n_p
    if L * max(n_p, n_q) >= 1 << 32:
        pytest.skip("refused")
    n_max, fast = max(n_p, n_q), L <= 64
    pos_p, pos_q, rec = L * n_p, L * n_q, L * min(n_p, n_q)
    find, chunks = L * ((n_p + 255) // 256), (rec + 127) // 128
    bps, krow, k = (n_max + 2047) // 2048, 512 if long_rows else 64, 8
    counts = L * 256 * bps
    hash_ws = L * k * (krow + 4) + 512 + L * n_max * 16 if fast else 0
    widened = L * k * (krow // 2) * 8
    sort_ws = max(4 * (4 * L * n_max + 256) + 4 * counts + 4 * L * 256 * ((bps + 63) // 64)
                  + L * 1024 + 1024, find * 24)
    fp = 16 * ((min(L, 64) + 15) // 16) if L > 1 else 0
    partials = 8 * (max(find, chunks) // 4096 + 2)
    for own, held in ((0, 8 * 1808), (min(n_p * n_q, 4 << 20), 4096 * 1808)):
        vals = [n_p, n_q, L, int(self_join), krow, 4, fp, hash_ws, widened, sort_ws, find, rec,
                chunks, partials, own, held, 256]
        out = (ctypes.c_uint64 * len(NAMES))()
        lib.layout((ctypes.c_uint64 * len(vals))(*vals), out)
        at = dict(zip(NAMES, out))
        size = dict(row_p=n_p * krow, norm_p=4 * n_p, key_p=8 * pos_p, perm_p=4 * pos_p,
                    sorted_p=8 * pos_p, list_p=4 * pos_p, tag_p=pos_p, fp_p=fp * n_p,
                    counters=64, partials=partials, hash_ws=hash_ws, widened=widened,
                    sort_ws=sort_ws, found=4096 * find, n_found=4 * find, found_off=8 * find,
                    rec_t=4 * rec, rec_pq=16 * rec, n_desc=4 * chunks, n_tile=4 * chunks,
                    desc_off=8 * chunks, tile_off=8 * chunks, desc_info=16 * rec,
                    desc_pq=16 * rec, own=8 * own, n_held=4 * 256, next=8 * 256,
                    held=at["held_bytes"])
        assert at["held_bytes"] >= held
        for q in ("row", "norm", "key", "perm", "sorted", "list", "tag", "fp"):
            if self_join:
                assert at[q + "_q"] == at[q + "_p"]
            else:
                size[q + "_q"] = size[q + "_p"] // n_p * n_q
        for a in size:
            assert at[a] % 256 == 0 and at[a] + size[a] <= at["total"], a
            for b in size:
                (a0, a1), (b0, b1) = LIVE.get(a, (0, 5)), LIVE.get(b, (0, 5))
                if a < b and a0 <= b1 and b0 <= a1:
                    assert at[a] + size[a] <= at[b] or at[b] + size[b] <= at[a], (a, b)
        if own == 0:
            per_pos = pos_p if self_join else pos_p + pos_q
            rows = n_p if self_join else n_p + n_q
            before = (rows * (krow + 4) + 20 * per_pos      # copies, norms; keys, sorted, perm
                      + rows * (16 if long_rows else 128)   # fingerprints or row records
                      + 24 * pos_p + 60 * rec + 24 * chunks # marks, sizes; records, tiles
                      + 16 * L * n_max + 12 * counts        # sort
                      + hash_ws + widened + 8 * pos_p // 4096 + 12 * 256 + held)
            # apart from rounding: to 256 bytes, and found buckets to whole blocks of 256
            assert at["total"] <= before + 256 * len(NAMES) + 4096 * 2 * L * (n_max < 4096)


@pytest.mark.parametrize("n", [1, 2, 255, 256, 1000, 1 << 31, (1 << 31) + 300, (1 << 32) - 1])
def test_run_end(lib, n):
    """Ends of runs of equal keys of every length, up to the longest (all of 2^32 - 1
    positions) and from starts near the end."""
    ends = {1, 2, n // 3, n // 2, n - 1, n, min(n, 1 << 31), min(n, (1 << 31) + 256)}
    for end in (e for e in ends if 0 < e <= n):
        for first in {0, end // 2, end - 1}:
            for p in {first + 1, first + (end - first) // 2, end}:
                if first < p <= end:
                    assert lib.run_end_of(first, end, p, n) == end, (first, end, p, n)


def test_block_entries(lib):
    for n in (1, 2047, 2048, 2049, (1 << 32) - 2048, (1 << 32) - 1):
        nb = (n + 2047) // 2048
        assert lib.entries(nb - 1, 2048, n) == n - 2048 * (nb - 1)
        assert lib.entries(0, 2048, n) == min(n, 2048)
