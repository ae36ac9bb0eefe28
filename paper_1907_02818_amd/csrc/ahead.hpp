// Which grids take the march of ahead3d.hpp, in which shape, and its launches.
#pragma once
#include "launch.hpp"
#include "tile3d.hpp"

namespace sadj {

// Small: 32 x 16 cells, 256 threads with two cells each, two workgroups per CU.  Wide: 16 bytes per lane, 512 threads: 64 x 16
// cells in fp64, 128 x 16 in fp32 (64 x 32 where rows are not whole vectors: one partial vector per row of 16 lanes), one
// workgroup per CU.  WideStream: Wide with streaming accesses to the arrays without reuse.
enum class AheadShape { None, Small, Wide, WideStream };

struct AheadPlan {
    AheadShape shape = AheadShape::None;
    int TX = 0, TY = 0;
    TileMap map{};
};

struct AheadArgs {
    March3dArgs m;              // arrays, extents and map, as the operation's other kernel takes them
    double w0, w[3][8];         // free-weight star: gather table (see StarArgs in star3d.hip)
};

// Grids whose arrays, `words` of them moved per call, take at most this many bytes.  Above, the kernels that keep the
// neighbours of a plane in L2 and stream the rest are as fast or faster: adjoint, this / those, fp64 384^3 (1.8 GB) radius 2
// 333 / 336 us, with u_prev_bar 519 / 492; 512^3 radius 4 742 / 703; 300 x 350 x 404 (1.4 GB) 274 / 292, radius 1 290 / 275.  Of 120
// drawn grids of 0.6 to 3 GB 45 lose, by up to 12 %; of 820 below the line 4, by up to 2.2 %.
constexpr double kAheadBytes = 560e6;
// Above this the 256 MB last-level cache does not serve enough of the repeated accesses, and streaming the others leaves it to
// c and r_bar: 0.82 to 0.95 of the time above 450 MB, 1.10 to 1.15 below 330 MB, equal within 2 % from 360 to 400.
constexpr double kAheadStreamBytes = 380e6;

// Small or Wide: the planes marched, times the relative cost of a step.  `beyond`: cheap planes of a chunk, counted as 2R full
// ones, which is what the z cut is planned with.  percent: cost of Small's step against Wide's.  Over 820 drawn grids this
// choice is 1.7 % (fp64) and 2.5 % (fp32) behind the better of the two; the grids are 1.43 and 1.40 times as fast as in the
// shapes of the other kernels.  Where Small's chunks are short (2R planes or less) the chip is hardly filled and its
// smaller workgroups win except at radius 1 in ragged fp32 rows (40^3 fp64 radius 4 4.3 us, Wide 5.3).
static inline AheadPlan plan_ahead(bool is_f64, int radius, int nx, int ny, int nz, int words, int percent, const int (&percent_short)[4],
                                   const LaunchOptions &opt)
{
    AheadPlan p;
    const double bytes = (double)nx * ny * nz * words * (is_f64 ? 8 : 4);
    if (opt.variant != 0 || opt.remainder != 0 || bytes > kAheadBytes) return p;
    // Rows that are no multiple of a cache line and fill tiles of 1 KB and more: where they are whole vectors such tiles run
    // (wide_tile_for_unaligned_rows); where not, those would fall back to one cell per lane, and the wide tile here is taken.
    const bool long_rows = wide_tile_for_unaligned_rows(nx, is_f64 ? 8 : 4, radius, !is_f64) != 0;
    if (long_rows && nx % (is_f64 ? 2 : 4) == 0) return p;
    const int wide_x = is_f64 ? 64 : nx % 4 == 0 ? 128 : 64, wide_y = !is_f64 && nx % 4 != 0 ? 32 : 16;
    // grid and type alone decide, so that options that move work between workgroups change nothing else
    TileMap small, wide;
    plan_march(small, nx, ny, nz, 32, 16, radius, LaunchOptions{}, 2);
    plan_march(wide, nx, ny, nz, wide_x, wide_y, radius, LaunchOptions{});
    if (small.tiles_a == 0 && small.zchunk <= 2 * radius)
        percent = percent_short[radius - 1];
    const bool is_small = !long_rows && percent * march_planes(small, 2 * radius, 2) < 100 * march_planes(wide, 2 * radius);
    p.shape = is_small ? AheadShape::Small : bytes > kAheadStreamBytes ? AheadShape::WideStream : AheadShape::Wide;
    p.TX = is_small ? 32 : wide_x;
    p.TY = is_small ? 16 : wide_y;
    p.map = is_small ? small : wide;
    if (opt.zchunk != 0 || opt.split != 0 || opt.xcd_map != 0 || opt.band != 0)
        plan_march(p.map, nx, ny, nz, p.TX, p.TY, radius, opt, is_small ? 2 : 1);
    return p;
}

// The wave adjoint; accumulates: u_prev_bar is read and written, writes_prev: written (or the array it replaces is).
static inline AheadPlan plan_adjoint_ahead(bool is_f64, int radius, int nx, int ny, int nz, bool accumulates, bool writes_prev,
                                           const LaunchOptions &opt)
{
    constexpr int short_f64[4] = {100, 99, 99, 99}, short_f32[4] = {74, 74, 74, 74}, short_ragged[4] = {100, 74, 74, 74}, both_f64[4] = {105, 105, 105, 105};
    const int words = accumulates ? 6 : writes_prev ? 5 : 4;
    if (is_f64) return plan_ahead(true, radius, nx, ny, nz, words, accumulates ? 105 : 115, accumulates ? both_f64 : short_f64, opt);
    return plan_ahead(false, radius, nx, ny, nz, words, 85, nx % 4 == 0 ? short_f32 : short_ragged, opt);
}

// opt.lds_pad > 0: dynamic LDS to request.
hipError_t launch_adjoint_wave3d_ahead(int is_f64, int radius, const AheadArgs &a, AheadShape shape, unsigned pad, hipStream_t stream);

}  // namespace sadj
