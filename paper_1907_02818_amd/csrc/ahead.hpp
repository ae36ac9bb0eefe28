// Which grids take the march of ahead3d.hpp, in which shape, and its launches.
#pragma once
#include "launch.hpp"
#include "tile3d.hpp"

namespace sadj {

// Rows, RowsStream: see plan_rows.  Small: 32 x 16 cells, 256 threads with two cells each, two workgroups per CU.  Wide: 16 bytes per lane, 512 threads: 64 x 16
// cells in fp64, 128 x 16 in fp32 (64 x 32 where rows are not whole vectors: one partial vector per row of 16 lanes), one
// workgroup per CU.  WideStream, RowsStream: with streaming accesses to the arrays without reuse.
enum class AheadShape { None, Small, Wide, WideStream, Rows, RowsStream };

// A tile of whole rows: bx vectors of 16 bytes by `by` rows, one per thread; h / bx is (h * reciprocal) >> 20 for h < 1024.  (Radii 3
// and 4 need more registers than 1024 threads have.)
constexpr int rows_threads(int radius) { return radius > 2 ? 512 : 1024; }
constexpr int rows_max_x(int radius) { return radius > 2 ? 128 : radius == 2 ? 256 : 512; }
constexpr int kRowsMaxY = 32;
struct RowsTile {
    int bx = 0, by = 0, reciprocal = 0;
};

// Wide and WideStream, `whole`: rows of whole vectors.
struct WideTile {
    int x, y;
};
static inline WideTile wide_tile(bool is_f64, bool whole) { return {is_f64 || !whole ? 64 : 128, is_f64 || whole ? 16 : 32}; }

struct AheadPlan {
    AheadShape shape = AheadShape::None;
    int TX = 0, TY = 0;
    RowsTile rows;
    TileMap map{};
};

struct AheadArgs {
    March3dArgs m;              // arrays, extents and map, as the operation's other kernel takes them
    double w0, w[3][8];         // free-weight star: gather table (see StarArgs in star3d.hip)
    RowsTile rows;              // of Rows and RowsStream
};

// When this march is taken, by the bytes a call moves (what it moves per cell, times the cells).  All figures: 1300 drawn grids
// of 3 10^4 to 1.2 10^8 cells, three sets of arrays in turn, time of the other kernels over time of this march; geometric mean
// (smallest).
//   limit    largest call.  Beyond it the kernels that keep the neighbours of a plane in L2 and stream the rest are as fast: wave
//            adjoint fp64 radius 4 560 .. 1400 MB 1.11 (1.06), radius 3 560 .. 800 MB 1.08, radius 1 560 .. 800 MB 0.97 (0.93); wave
//            primal radius 1 fp64 120 .. 250 MB 1.10 (0.98), 560 .. 800 MB 0.95, fp32 120 .. 250 MB 1.02 (0.93), 250 .. 560 MB 0.89
//            (0.70); star adjoint radius 2 to 4 560 .. 800 MB 1.05 to 1.13.
//   stream   largest call whose arrays without reuse go through the caches.  Arrays that the same loop touches in every step are
//            found in the 256 MB last-level cache up to 380 MB (fp64 200^3: 42 us cached, 56 streaming; 256^3: 96 and 84); a single
//            call finds less (wave adjoint fp64, three sets: 90 .. 120 MB 1.42 cached and 1.29 streaming, 130 .. 200 MB 1.13 and 1.24).
struct AheadRule {
    int words;                  // moved per cell
    double limit, stream;
    int percent;                // cost of Small's step against Wide's
    int percent_short;          // the same where Small's chunks are 2R planes or shorter and the chip is hardly filled
    bool long_rows_stay;        // rows that wide_tile_for_unaligned_rows gives tiles of 1 KB and more, in whole vectors, keep them
};
constexpr double kAheadLoopStream = 380e6, kAheadCallStream = 125e6;
constexpr int kPercentStream = 150;     // streaming, Wide against Small, which has no streaming form (12 of 455 such grids take Small)

// Tiles of whole rows, for rows that are no multiples of a cache line or fill the wide tiles badly: the rows of a tile are then one piece of memory, whose
// inner lines are used in full whatever the rows' alignment, and no thread lies beside the grid.  (Tiles of a fixed width start and end within lines
// on both sides, and the last one is in part outside the grid.)  A tile has as many rows as its threads allow.  Time in the tiles below and in those of
// the larger grids over time in these, 2876 drawn grids up to 3 GB that a call moves and this rule takes (geometric mean 1.18), 5 % of them below the
// second figure and 5 % above the third:
//   radius 1, 2, rows that are no whole vectors 0.91, 1.02, 1.61; other rows that are no whole lines 0.85, 0.99, 1.38; whole lines 0.90, 0.98, 1.26
//   radius 3, 4, the first and second of these 0.79, 1.01, 1.63 and 0.94, 1.00, 1.49
// Below 0.97 are 55 of them, half in calls of less than 170 MB, many of 32 rows; grids next to them in size are faster (fp64 573 x 60 x 360 0.93, 600 x 60 x 360 1.07).
// The bounds, with the same quotient beyond them:
//   bytes of a call, 125 MB (50 .. 125 MB: 0.86 to 1.23); radius 1, 257 to 512 vectors, where wide_tile_for_unaligned_rows finds no tile, and
//     radius 3 and 4: 250 MB (0.91 to 1.22 and 0.86 to 1.32)
//   vectors in a row: 256, radius 1 512 (where wide_tile_for_unaligned_rows finds a tile 0.99 to 1.15), radius 3 and 4 128, or four
//     rows a tile; with fewer every plane is read three times over (0.63 to 1.15); radius 4, whole vectors, six rows (0.95 to 1.15)
//   where the other choice is the march of small grids, vectors that this march computes over those of its Wide tiles, which shallow grids and grids of few
//     rows exceed: 0.7 for rows that fit a wide tile, which are whole there already (0.83 to 1.10, geometric mean of 67 grids 0.95); radius 1, 2, whole
//     vectors 1.3 (0.88 to 1.15, 0.96), in loops in the last-level cache 1.2 (0.93 to 1.04, 0.99), rows of whole lines, which gain
//     nothing from their alignment, 1.1 (0.91 to 1.07, 0.99)
//   rows of whole lines: wide tiles filled to less than 0.9 (else 0.85 to 1.19, 512^3 fp32 0.92; loops in the last-level cache 0.97 to 1.10)
//   fewer than 20 R planes: 0.95 to 1.17; they stay in the other tiles, as do fewer than 32 rows (not measured).
// fp32 500^3 radius 1 primal 389 -> 344 us; 300 x 350 x 404 radius 2 star adjoint 164 -> 122; 1000 x 300 x 404 primal 460 -> 368.
static inline bool plan_rows(AheadPlan &p, bool is_f64, int radius, int nx, int ny, int nz, double bytes, const AheadRule &rule, LaunchOptions opt)
{
    const int size = is_f64 ? 8 : 4, px = 16 / size, bx = cdiv_i(nx, px), threads = rows_threads(radius);
    const bool whole = nx % px == 0, lines = (long)nx * size % 128 == 0;
    const WideTile wide = wide_tile(is_f64, whole);
    if (bx < threads / kRowsMaxY || bx > rows_max_x(radius) || ny < 32 || nz < 20 * radius) return false;
    if (bx > 256 && wide_tile_for_unaligned_rows(nx, size, radius, !is_f64) != 0) return false;
    if (bytes <= (radius > 2 || bx > 256 ? 250e6 : kAheadCallStream)) return false;
    if (radius == 4 && whole && threads / bx < 6) return false;
    if (lines && (radius > 2 || bx > 256 || bytes <= rule.stream || 10L * nx >= 9L * cdiv_i(nx, wide.x) * wide.x)) return false;
    const double most = 0x1p31 / ((double)nx * ny * size) - 16;                // planes of a chunk, see MarchedArray
    if (most < 32) return false;                                               // planes of more than 44.7 MB
    const RowsTile rows = {bx, cdiv_i(ny, cdiv_i(ny, threads / bx)), (1 << 20) / bx + 1};
    TileMap map;
    plan_march(map, nx, ny, nz, bx * px, rows.by, radius, LaunchOptions{});    // grid and type alone decide, as in plan_ahead
    const int percent = nx <= wide.x ? 70 : radius > 2 || !whole ? 0 : lines ? 110 : bytes > rule.stream ? 130 : 120;
    if (percent != 0 && bytes <= rule.limit) {                                 // a step of Wide has 512 vectors
        TileMap other;
        plan_march(other, nx, ny, nz, wide.x, wide.y, radius, LaunchOptions{});
        if (100L * threads * march_planes(map, 2 * radius) > 512L * percent * march_planes(other, 2 * radius)) return false;
    }
    if (opt.zchunk != 0 || opt.split != 0 || opt.xcd_map != 0 || opt.band != 0) plan_march(map, nx, ny, nz, bx * px, rows.by, radius, opt);
    if (map.zchunk > most || map.zchunk_a > most) {
        opt.zchunk = cdiv_i(nz, cdiv_i(nz, (int)most));
        plan_march(map, nx, ny, nz, bx * px, rows.by, radius, opt);
    }
    p.shape = bytes > rule.stream ? AheadShape::RowsStream : AheadShape::Rows;
    p.TX = bx * px;
    p.TY = rows.by;
    p.rows = rows;
    p.map = map;
    return true;
}

// Small or Wide: the planes marched, times the relative cost of a step.  The cheap planes of a chunk count as 2R full ones, which
// is also what the z cut is planned with (other weights moved no grid's time by more than 3 %).
static inline AheadPlan plan_ahead(bool is_f64, int radius, int nx, int ny, int nz, const AheadRule &rule, const LaunchOptions &opt)
{
    AheadPlan p;
    const double bytes = (double)nx * ny * nz * rule.words * (is_f64 ? 8 : 4);
    if (opt.variant != 0 || opt.remainder != 0 || opt.ahead != 0) return p;
    if (plan_rows(p, is_f64, radius, nx, ny, nz, bytes, rule, opt)) return p;
    if (bytes > rule.limit) return p;
    const bool whole = nx % (is_f64 ? 2 : 4) == 0;
    const bool long_rows = rule.long_rows_stay && wide_tile_for_unaligned_rows(nx, is_f64 ? 8 : 4, radius, !is_f64) != 0;
    if (long_rows && whole) return p;
    const WideTile wide_shape = wide_tile(is_f64, whole);
    // grid and type alone decide, so that options that move work between workgroups change nothing else
    TileMap small, wide;
    plan_march(small, nx, ny, nz, 32, 16, radius, LaunchOptions{}, 2);
    plan_march(wide, nx, ny, nz, wide_shape.x, wide_shape.y, radius, LaunchOptions{});
    const bool stream = bytes > rule.stream;
    const int percent = small.tiles_a == 0 && small.zchunk <= 2 * radius ? rule.percent_short : stream ? kPercentStream : rule.percent;
    const bool is_small = !long_rows && percent * march_planes(small, 2 * radius, 2) < 100 * march_planes(wide, 2 * radius);
    p.shape = is_small ? AheadShape::Small : stream ? AheadShape::WideStream : AheadShape::Wide;
    p.TX = is_small ? 32 : wide_shape.x;
    p.TY = is_small ? 16 : wide_shape.y;
    p.map = is_small ? small : wide;
    if (opt.zchunk != 0 || opt.split != 0 || opt.xcd_map != 0 || opt.band != 0)
        plan_march(p.map, nx, ny, nz, p.TX, p.TY, radius, opt, is_small ? 2 : 1);
    return p;
}

// The wave adjoint; accumulates: u_prev_bar is read and written, writes_prev: written (or the array it replaces is), loop: a step
// of a time loop that starts from the r_bar of the step before (launch_adjoint_wave3d_middle).  The first two steps of a loop and the
// single steps between fused passes count as lone calls.  Below 120 MB 1.42 to 1.45 (fp64) and 1.40 (fp32) times as fast as in the tiles of
// wave3d_adjoint.hip, 1 % behind the better of the two shapes.  40^3 fp64 radius 4, Small / Wide: 4.3 / 5.3 us; 80 x 96 x 112 with
// u_prev_bar 11.7 / 10.2.
static inline AheadPlan plan_adjoint_ahead(bool is_f64, int radius, int nx, int ny, int nz, bool accumulates, bool writes_prev, bool loop,
                                           const LaunchOptions &opt)
{
    const int words = accumulates ? 6 : writes_prev ? 5 : 4;
    const double limit = radius == 4 ? 1400e6 : radius == 3 ? 800e6 : 560e6, stream = loop ? kAheadLoopStream : kAheadCallStream;
    AheadRule rule{words, limit, stream, 85, 74, true};
    if (is_f64) rule = {words, limit, stream, accumulates ? 105 : 115, accumulates ? 105 : radius == 1 ? 100 : 99, true};
    else if (radius == 1 && nx % 4 != 0) rule.percent_short = 100;
    return plan_ahead(is_f64, radius, nx, ny, nz, rule, opt);
}

// The free-weight star, both directions, and the wave primal.  Below 120 MB star adjoint 1.46 (fp64) and 1.51 (fp32) times as
// fast as before, star primal 1.63 and 1.56, wave primal 1.59 and 1.82.
static inline AheadPlan plan_star_ahead(bool is_f64, int radius, int nx, int ny, int nz, bool adjoint, bool wave, LaunchOptions opt)
{
    opt.remainder = 0;                               // an option of the wave adjoint
    const int percent = is_f64 ? (wave ? 115 : 110) : adjoint ? 80 : 70;
    const double limit = radius == 4 ? 1400e6 : radius > 1 ? (adjoint ? 800e6 : 560e6) : adjoint ? 560e6 : is_f64 ? 250e6 : kAheadCallStream;
    const AheadRule rule{adjoint || wave ? 4 : 3, limit, kAheadCallStream, percent, percent, false};
    return plan_ahead(is_f64, radius, nx, ny, nz, rule, opt);
}

// pad: dynamic LDS to request.
static inline unsigned ahead_pad(const LaunchOptions &opt) { return opt.lds_pad > 0 ? (unsigned)opt.lds_pad : 0u; }
hipError_t launch_adjoint_wave3d_ahead(int is_f64, int radius, const AheadArgs &a, AheadShape shape, unsigned pad, hipStream_t stream);
hipError_t launch_primal_wave3d_ahead(int is_f64, int radius, const AheadArgs &a, AheadShape shape, unsigned pad, hipStream_t stream);
hipError_t launch_star3d_ahead(int adjoint, int is_f64, int radius, const AheadArgs &a, AheadShape shape, unsigned pad, hipStream_t stream);

}  // namespace sadj
