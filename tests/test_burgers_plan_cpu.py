"""CPU test of the launch order of the Burgers time loops (csrc/burgers_plan.hpp): a driver compiled with
the host compiler replays every launch on rows that hold the number of the state (or adjoint) they
contain, and checks that each launch finds what it reads, that no launch writes what it reads, that
rows stay inside the caller's arrays, and that the results end where the header says."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

DRIVER = r"""
#include "burgers_plan.hpp"
#include <cstdio>
#include <cstdlib>
#include <initializer_list>
#include <vector>

// One "row" is one byte of a flat buffer; val[i] says what row i holds: state t = t, adjoint of
// state t = 1000000 + t, unknown = -1.
static std::vector<int> val;
static std::vector<char> given;            // rows no launch may write
static char arena[4096];
static int checkpoint_every, failures, most = sadj::kRecomputeSteps;
static long top;
#define NEED(c) do { if (!(c)) { if (failures++ < 5) std::printf("line %d: %s\n", __LINE__, #c); return 1; } } while (0)

static long at(const char *p) { return p - arena; }

struct Ops {
    int launches = 0;
    int put(char *p, int v) { long i = at(p); NEED(i >= 0 && i < top && !given[i]); val[i] = v; return 0; }
    int forward(const char *src, char *rows, long first, long every, int m, char *last, bool hold)
    {
        ++launches;
        NEED(m >= 1 && m <= sadj::kForwardSteps && first >= 1 && every >= 1);
        long i = at(src);
        NEED(i >= 0 && i < top && val[i] >= 0 && val[i] < 1000000);
        NEED(hold || (first == 1 && every == 1 && !last));
        const int t = val[i];
        long next = first;
        for (int s = 1; s <= m; ++s)
            if (s == next) { NEED(rows != src); if (put(rows, t + s)) return 1; rows += 1; next += every; }
        if (last) { NEED(last != src); if (put(last, t + m)) return 1; }
        return 0;
    }
    int reverse(const char *src, const char *rows, int first, int every, int m, const char *in, char *out)
    {
        ++launches;
        NEED(m >= 1 && m <= (every == 1 ? sadj::kReverseSteps : most));
        NEED(in != out && out != src);
        long i = at(src);
        NEED(i >= 0 && i < top && val[i] >= 0 && val[i] < 1000000);
        const int t = val[i];
        int next = first;
        for (int s = 1; s < m; ++s)
            if (s == next) { NEED(at(rows) >= 0 && at(rows) < top && val[at(rows)] == t + s && rows != out); rows += 1; next += every; }
        NEED(val[at(in)] == 1000000 + t + m);
        return put(out, 1000000 + t);
    }
    int reverse_first(const char *u, const char *in, char *out)
    {
        ++launches;
        NEED(val[at(u)] >= 0 && val[at(in)] == 1000000 + val[at(u)] + 1);
        return put(out, 1000000 + val[at(u)]);
    }
};

static void reset(long rows) { top = rows; val.assign(rows, -1); given.assign(rows, 0); }

static int history(long nsteps)
{
    Ops ops;
    reset(nsteps + 3);
    val[0] = 0; given[0] = 1;
    if (sadj::plan_burgers_history_forward(ops, arena, 1, nsteps)) return 1;
    for (long t = 0; t <= nsteps; ++t) NEED(val[t] == t);
    NEED(ops.launches == (nsteps + sadj::kForwardSteps - 1) / sadj::kForwardSteps);
    for (long t = 0; t <= nsteps; ++t) given[t] = 1;
    char *lam[2] = {arena + nsteps + 1, arena + nsteps + 2};
    val[nsteps + 1] = 1000000 + nsteps;
    char *const l[2] = {lam[0], lam[1]};
    if (sadj::plan_burgers_history_reverse(ops, arena, 1, nsteps, l)) return 1;
    NEED(val[nsteps + 1 + nsteps % 2] == 1000000);
    return 0;
}

static int ckpt(long nsteps, long every, bool want_final)
{
    Ops ops;
    const long rows = nsteps / every + 1, work = rows, fin = work + 2;
    reset(fin + 1);
    val[0] = 0; given[0] = 1;
    if (sadj::plan_burgers_ckpt_forward(ops, arena, arena + work, want_final ? arena + fin : nullptr, 1, nsteps, every)) return 1;
    for (long j = 0; j < rows; ++j) NEED(val[j] == j * every);
    if (want_final && nsteps > 0) NEED(val[fin] == nsteps);
    if (every == 1) return 0;
    // reverse: exactly the arrays the call is documented to take
    const long need = (nsteps > 0 ? nsteps - 1 : 0) / every + 1;
    reset(need + every - 1 + 2);
    for (long j = 0; j < need; ++j) { val[j] = (int)(j * every); given[j] = 1; }
    char *const lam[2] = {arena + need + every - 1, arena + need + every};
    val[at(lam[0])] = 1000000 + nsteps;
    sadj::BurgersCkptReverse<Ops> plan{ops, arena, arena + need, 1, every, most};
    if (plan.run(nsteps, lam)) return 1;
    NEED(val[at(lam[nsteps % 2])] == 1000000);
    return 0;
}

// The longest pass of a checkpointed sweep is 8, 12 or 16 steps, whichever costs least (window: 256 or 512 cells in long arrays, 128 else).
static int longest_pass()
{
    for (long n = 3; n < (1L << 30); n = n * 3 / 2 + 1)
        for (int window : {128, 256, 512})
            for (long every = 2; every <= 100; ++every) {
                const int m = sadj::recompute_steps(n, window, every);
                NEED(m == 8 || m == 12 || m == 16);
                NEED(sadj::recompute_kernel(m) == m);
            }
    NEED(sadj::recompute_steps(3000001, 256, 16) == 16 && sadj::recompute_steps(17000000, 256, 16) == 16);
    NEED(sadj::recompute_steps(6000000, 256, 8) == 8 && sadj::recompute_steps(1200000, 256, 6) == 12);
    NEED(sadj::recompute_steps(3000000, 512, 16) == 16 && sadj::recompute_steps(1000000, 512, 12) == 12);
    NEED(sadj::recompute_steps(8000000, 512, 8) == 8 && sadj::recompute_steps(100000, 128, 16) == 16);
    return 0;
}

int main()
{
    if (longest_pass()) std::printf("longest pass\n");
    for (int steps : {8, 12, 16}) {
        most = steps;
        for (long n = 0; n <= 150; ++n) {
            if (steps == 16 && history(n)) std::printf("history %ld\n", n);
            for (long every = 1; every <= 70; ++every)
                for (int f = 0; f < 2; ++f)
                    if (ckpt(n, every, f)) std::printf("ckpt nsteps %ld every %ld most %d\n", n, every, most);
        }
        for (long n : {1000L, 1001L, 2047L, 2048L}) {
            if (steps == 16 && history(n)) std::printf("history %ld\n", n);
            for (long every : {1L, 2L, 7L, 8L, 9L, 16L, 17L, 33L, 100L, 1500L})
                if (ckpt(n, every, true)) std::printf("ckpt nsteps %ld every %ld most %d\n", n, every, most);
        }
    }
    std::printf("failures %d\n", failures);
    return failures != 0;
}
"""


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src = d / "driver.cpp"
    src.write_text(DRIVER)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-I", os.path.join(ROOT, "paper_1907_02818_amd", "csrc"), str(src), "-o",
                           str(d / "driver")])
    return str(d / "driver")


def test_every_launch_finds_what_it_reads_and_the_results_end_in_place(driver):
    p = subprocess.run([driver], stdout=subprocess.PIPE, text=True)
    assert p.returncode == 0, p.stdout
