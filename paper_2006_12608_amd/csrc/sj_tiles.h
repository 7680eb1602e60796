// sj_tiles.h -- the order in which the K-streamed kernel's workgroups take the
// 256 x 256 tiles of the result (index arithmetic only, for device and host).
#pragma once

#include <stdint.h>

#if defined(__HIPCC__)
#define SJ_HD __host__ __device__ __forceinline__
#else
#define SJ_HD inline
#endif

namespace sjk {

// Tile numbers: groups of ST_G x ST_G tiles, row-major over the groups and inside
// each, so that workgroups running at once share their operand rows in L2.
// Numbers have no gaps where groups at the edges are smaller or, in a self-join's
// triangle (TRI: n_pt == n_qt, tiles pt <= qt only), lie on or below the diagonal:
// workgroup b takes the tiles numbered b, b + step, ..., and a number left out
// would fall to the same workgroups in every group.  With the triangle's skipped
// tiles numbered too, the busiest of 256 workgroups had 12 tiles of 16384 rows
// where the mean is 8.1: a call on bf16 rows of 2048 bytes took 302 us, without gaps
// 264 (int8 rows of 1024: 185 and 155).
constexpr uint32_t ST_G = 8;

struct TileAt {
    uint32_t pt, qt;
};

template <bool TRI>
struct TileWalk {
    uint32_t n_pt, n_qt, idx, step, gp = 0;

    SJ_HD TileWalk(uint32_t n_pt_, uint32_t n_qt_, uint32_t first, uint32_t step_)
        : n_pt(n_pt_), n_qt(n_qt_), idx(first), step(step_)
    {
    }
    // Tiles in all (below 2^31 for every launch).
    static SJ_HD uint32_t count(uint32_t n_pt, uint32_t n_qt)
    {
        return TRI ? (uint32_t)((uint64_t)n_pt * (n_pt + 1) / 2) : n_pt * n_qt;
    }
    // The triangle's tiles in the (whole) group rows before gp: each has its
    // diagonal group's ST_G (ST_G + 1) / 2 and ST_G for every tile column after it.
    SJ_HD uint32_t tri_first(uint32_t g) const
    {
        return g * (ST_G * n_pt + ST_G / 2 - ST_G * ST_G / 2 * g);
    }
    // The next tile; false past the last.
    SJ_HD bool next(TileAt &x)
    {
        if (idx >= count(n_pt, n_qt))
            return false;
        if constexpr (TRI) {
            while (ST_G * (gp + 1) < n_pt && idx >= tri_first(gp + 1))
                ++gp;
            uint32_t r = idx - tri_first(gp);
            const uint32_t p0 = gp * ST_G;
            const uint32_t hp = n_pt - p0 < ST_G ? n_pt - p0 : ST_G, diag = hp * (hp + 1) / 2;
            if (r < diag) {
                uint32_t i = 0;   // row i of the diagonal group holds hp - i tiles
                while (r >= hp - i)
                    r -= hp - i++;
                x = {p0 + i, p0 + i + r};
            } else {
                r -= diag;
                const uint32_t gq = gp + 1 + r / (hp * ST_G), in = r % (hp * ST_G);
                const uint32_t q0 = gq * ST_G, hq = n_pt - q0 < ST_G ? n_pt - q0 : ST_G;
                x = {p0 + in / hq, q0 + in % hq};
            }
        } else {
            const uint32_t g = idx / (ST_G * n_qt), r = idx - g * (ST_G * n_qt);
            const uint32_t p0 = g * ST_G, hp = n_pt - p0 < ST_G ? n_pt - p0 : ST_G;
            const uint32_t gq = r / (hp * ST_G), in = r - gq * (hp * ST_G);
            const uint32_t q0 = gq * ST_G, hq = n_qt - q0 < ST_G ? n_qt - q0 : ST_G;
            x = {p0 + in / hq, q0 + in % hq};
        }
        idx += step;   // (both below 2^31: no wrap)
        return true;
    }
};

}  // namespace sjk
