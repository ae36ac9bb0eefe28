// Which tile shape a 3-D kernel takes for a grid.  Host code without any device call, so that the rules can be
// checked on a CPU.
#pragma once
#include <cstddef>
#include <cstdint>

namespace sadj {

static inline int cdiv_i(int a, int b) { return (a + b - 1) / b; }

// Rows whose length in bytes is not a multiple of the 128-byte cache line (nx = 1000 in fp64:
// every other row starts in the middle of a line).  Tile rows then begin and end inside a line
// on most rows, and tiles with long rows (fewer row ends per byte) measured faster than the
// default shapes, while for line-aligned rows they measured equal or slower.
//
// Radius 1 keeps three running sums per cell, so eight cells per lane fit the register file:
// tiles of 256 (fp32 wave kernels: 512) cells x 16 rows measured 4-10 points faster (500^3, 1000^3,
// 200 x 700 x 1500, both dtypes, adjoint and primal).  Larger radii stay at four fp64 (eight
// fp32) cells per lane and trade tile rows for width: 1 KB x 16 rows instead of 512 B x 32
// (radius 4 fp64 at 500^3, 1000^3, 250 x 900 x 1100, 300 x 300 x 1250: adjoint +2 to +5
// points, with u_prev_bar +3 to +7, primal +3 to +6).
//
// Returns the tile width in cells to use, or 0 for the default shape; a width qualifies if its
// tiles cover nx with at most 10 % idle columns.
static inline int wide_tile_for_unaligned_rows(int nx, size_t elem_bytes, int radius, bool allow_512)
{
    if (((size_t)nx * elem_bytes) % 128 == 0) return 0;
    auto fills = [nx](int tx) { return 10L * nx >= 9L * cdiv_i(nx, tx) * tx; };
    if (radius == 1) {
        if (allow_512 && fills(512)) return 512;
        return fills(256) ? 256 : 0;
    }
    const int tx = (int)(1024 / elem_bytes);
    return fills(tx) ? tx : 0;
}

// Shape of the wave primal (numbered as the adjoint's, option "wave3d.variant"); addresses: those of all arrays,
// or-ed together.  512-cell tiles move four fp32 cells per lane and need whole 16-byte vectors (500^3: 398 -> 389 us);
// where rows or arrays are whole 8-byte vectors only, 256-cell tiles with two cells per lane stay the choice
// (266 x 258 x 510 98 us, one cell per lane, which the wider tile would fall back to, 140; 197 x 78 x 1022 45 and 71).
static inline long primal_shape(size_t elem_bytes, int radius, int nx, uintptr_t addresses)
{
    const bool whole = nx % 4 == 0 && addresses % 16 == 0;
    const int wide = wide_tile_for_unaligned_rows(nx, elem_bytes, radius, elem_bytes == 4 && radius == 1 && whole);
    if (radius == 1 && wide == 512) return 11;
    if (radius == 1 && wide == 256) return 10;
    if (radius > 1 && wide) return 5;
    return elem_bytes == 8 ? 3 : 8;              // measured best per dtype
}

}  // namespace sadj
