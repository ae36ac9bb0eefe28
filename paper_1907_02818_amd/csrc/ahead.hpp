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

// Small or Wide: the planes marched, times the relative cost of a step.  The cheap planes of a chunk count as 2R full ones, which
// is also what the z cut is planned with (other weights moved no grid's time by more than 3 %).
static inline AheadPlan plan_ahead(bool is_f64, int radius, int nx, int ny, int nz, const AheadRule &rule, const LaunchOptions &opt)
{
    AheadPlan p;
    const double bytes = (double)nx * ny * nz * rule.words * (is_f64 ? 8 : 4);
    if (opt.variant != 0 || opt.remainder != 0 || opt.ahead != 0 || bytes > rule.limit) return p;
    const bool whole = nx % (is_f64 ? 2 : 4) == 0;
    const bool long_rows = rule.long_rows_stay && wide_tile_for_unaligned_rows(nx, is_f64 ? 8 : 4, radius, !is_f64) != 0;
    if (long_rows && whole) return p;
    const int wide_x = is_f64 ? 64 : whole ? 128 : 64, wide_y = !is_f64 && !whole ? 32 : 16;
    // grid and type alone decide, so that options that move work between workgroups change nothing else
    TileMap small, wide;
    plan_march(small, nx, ny, nz, 32, 16, radius, LaunchOptions{}, 2);
    plan_march(wide, nx, ny, nz, wide_x, wide_y, radius, LaunchOptions{});
    const bool stream = bytes > rule.stream;
    const int percent = small.tiles_a == 0 && small.zchunk <= 2 * radius ? rule.percent_short : stream ? kPercentStream : rule.percent;
    const bool is_small = !long_rows && percent * march_planes(small, 2 * radius, 2) < 100 * march_planes(wide, 2 * radius);
    p.shape = is_small ? AheadShape::Small : stream ? AheadShape::WideStream : AheadShape::Wide;
    p.TX = is_small ? 32 : wide_x;
    p.TY = is_small ? 16 : wide_y;
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
