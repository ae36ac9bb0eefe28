"""CPU test of the plans of the 3-D march with requests ahead (csrc/ahead.hpp): a grid that is not left to the other tiles
gets workgroups that cover each tile and plane once, with chunks whose byte offsets stay below 2^31, for every operation, radius,
type and extent up to planes of 2^28 cells; and tiles of whole rows are not taken where they measured slower."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

DRIVER = r"""
#include "ahead.hpp"
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <vector>
using namespace sadj;

static int failures, taken, rows, cut, refused, zchunk;
static void check(const AheadPlan &p, const char *op, bool f64, int R, int nx, int ny, int nz)
{
    const char *what = nullptr;
    const double plane = (double)nx * ny * (f64 ? 8 : 4);
    if (p.shape == AheadShape::None) { refused += plane >= 0x1p31 / 48; return; }
    ++taken;
    const TileMap &m = p.map;
    const bool whole_rows = p.shape == AheadShape::Rows || p.shape == AheadShape::RowsStream;
    rows += whole_rows;
    cut += whole_rows && zchunk >= nz && (nz + 16) * plane > 0x1p31;           // one chunk was asked for and is too long
    if (m.total_blocks < 1) what = "no workgroups";
    else if ((long)m.ntx * p.TX < nx || (long)m.nty * p.TY < ny) what = "cells without a tile";
    else if (whole_rows && (m.ntx != 1 || p.rows.bx * p.rows.by > rows_threads(R) || p.rows.by > kRowsMaxY)) what = "tile of whole rows";
    std::vector<int> at((size_t)m.ntx * m.nty, 0), planes((size_t)m.ntx * m.nty, 0);
    int longest = 0;
    for (int pass = 0; !what && pass < 2; ++pass)
        for (int b = 0; b < m.total_blocks; ++b) {
            int tix, tiy, zs, ze;
            block_to_tile(m, b, tix, tiy, zs, ze);
            if (tix < 0 || tix >= m.ntx || tiy < 0 || tiy >= m.nty || zs < 0 || ze > nz || zs >= ze) { what = "range of a workgroup"; break; }
            planes[(size_t)tiy * m.ntx + tix] += pass == 0 ? ze - zs : 0;
            if (zs == 0) ++at[(size_t)tiy * m.ntx + tix];
            if (ze - zs > longest) longest = ze - zs;
        }
    for (size_t i = 0; !what && i < at.size(); ++i)
        if (at[i] != 2 || planes[i] != nz) what = "planes covered";
    if (!what && (longest + 16) * plane > 0x1p31) what = "offsets of a chunk";
    if (what && failures++ < 8) std::printf("%s: %s f64=%d R=%d nz=%d ny=%d nx=%d\n", what, op, (int)f64, R, nz, ny, nx);
}

static void all(int nx, int ny, int nz, const LaunchOptions &opt)
{
    zchunk = opt.zchunk;
    for (int f64 = 0; f64 < 2; ++f64)
        for (int R = 1; R <= 4; ++R) {
            if (nx < 2 * R + 1 || ny < 2 * R + 1 || nz < 2 * R + 1) continue;
            check(plan_adjoint_ahead(f64, R, nx, ny, nz, false, false, false, opt), "adjoint", f64, R, nx, ny, nz);
            check(plan_adjoint_ahead(f64, R, nx, ny, nz, true, true, false, opt), "adjoint, u_prev_bar", f64, R, nx, ny, nz);
            check(plan_adjoint_ahead(f64, R, nx, ny, nz, false, true, true, opt), "loop", f64, R, nx, ny, nz);
            check(plan_star_ahead(f64, R, nx, ny, nz, true, false, opt), "star adjoint", f64, R, nx, ny, nz);
            check(plan_star_ahead(f64, R, nx, ny, nz, false, false, opt), "star primal", f64, R, nx, ny, nz);
            check(plan_star_ahead(f64, R, nx, ny, nz, false, true, opt), "wave primal", f64, R, nx, ny, nz);
        }
}

static bool in_whole_rows(const AheadPlan &p) { return p.shape == AheadShape::Rows || p.shape == AheadShape::RowsStream; }
#define NEED(c) do { if (!(c) && failures++ < 8) std::printf("%s\n", #c); } while (0)

// grids measured slower (0.83 to 0.93 times as fast) and faster (1.1 to 1.6 times) in tiles of whole rows
static void choices()
{
    const LaunchOptions opt;
    NEED(!in_whole_rows(plan_adjoint_ahead(true, 4, 43, 499, 300, true, true, false, opt)));
    NEED(!in_whole_rows(plan_adjoint_ahead(false, 4, 100, 508, 448, false, false, false, opt)));
    NEED(!in_whole_rows(plan_adjoint_ahead(true, 3, 55, 291, 423, true, true, false, opt)));
    NEED(!in_whole_rows(plan_star_ahead(true, 2, 382, 327, 64, true, false, opt)));
    NEED(!in_whole_rows(plan_star_ahead(true, 2, 336, 224, 81, true, false, opt)));
    NEED(!in_whole_rows(plan_star_ahead(true, 1, 424, 544, 32, false, true, opt)));
    NEED(!in_whole_rows(plan_star_ahead(true, 2, 298, 790, 41, false, false, opt)));
    NEED(!in_whole_rows(plan_adjoint_ahead(true, 1, 63, 214, 608, false, false, false, opt)));
    NEED(in_whole_rows(plan_star_ahead(true, 1, 386, 32, 336, true, false, opt)));
    NEED(in_whole_rows(plan_adjoint_ahead(true, 1, 350, 109, 188, true, true, false, opt)));
    NEED(in_whole_rows(plan_adjoint_ahead(true, 2, 350, 121, 160, false, true, true, opt)));
    NEED(in_whole_rows(plan_adjoint_ahead(false, 2, 192, 236, 170, true, true, false, opt)));
    NEED(in_whole_rows(plan_star_ahead(false, 1, 500, 500, 500, false, true, opt)));
    NEED(in_whole_rows(plan_star_ahead(false, 2, 404, 350, 300, true, false, opt)));
    NEED(in_whole_rows(plan_adjoint_ahead(false, 2, 390, 110, 590, true, true, false, opt)));
    NEED(in_whole_rows(plan_adjoint_ahead(false, 4, 107, 931, 652, false, true, true, opt)));
}

int main()
{
    choices();
    LaunchOptions opt, chunk, split;
    chunk.zchunk = 1000;
    split.split = 1;
    // just below and above the largest plane that whole rows take (2^31 / 48 bytes)
    const int grids[][3] = {{500, 12000, 20}, {510, 10900, 20}, {510, 11000, 20}, {510, 11000, 100}, {900, 7000, 24}, {1002, 13000, 24},
                            {1022, 11500, 40}, {1001, 12000, 40}, {500, 12000, 40}, {500, 12000, 81}, {341, 16500, 80}, {16384, 16384, 9}};
    for (const auto &g : grids) { all(g[0], g[1], g[2], opt); all(g[0], g[1], g[2], chunk); }
    std::srand(7);
    auto extent = [](double lo, double hi) { return (int)std::lround(lo * std::pow(hi / lo, std::rand() / (double)RAND_MAX)); };
    for (int i = 0; i < 6000; ++i) {
        const int nx = extent(3, i % 2 ? 2048 : 1 << 20), ny = extent(3, std::fmax(3, 0x1p28 / nx));
        const int nz = extent(3, std::fmin(std::fmax(3, 4e9 / ((double)nx * ny)), 4e4));
        all(nx, ny, nz, i % 3 == 0 ? chunk : i % 3 == 1 ? split : opt);
    }
    std::printf("taken %d, whole rows %d, chunks cut %d, large planes left to the other tiles %d\n", taken, rows, cut, refused);
    return failures != 0 || taken < 10000 || rows < 1000 || cut < 100 || refused < 1000;
}
"""


def test_every_plan_covers_its_grid_once(tmp_path):
    src = tmp_path / "driver.hip"
    src.write_text(DRIVER)
    subprocess.check_call([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-host-only", "-std=c++17", "-O2", "-I",
                           os.path.join(ROOT, "paper_1907_02818_amd", "csrc"), str(src), "-o", str(tmp_path / "driver")])
    p = subprocess.run([str(tmp_path / "driver")], stdout=subprocess.PIPE, text=True)
    assert p.returncode == 0, p.stdout
