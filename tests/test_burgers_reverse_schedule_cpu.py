"""CPU test of the order of requests and steps of a reverse pass of the Burgers time loop over stored states
(csrc/burgers_plan.hpp): every state is requested once and no other, early enough and never into a register
set that still waits for its step; and of the lengths into which a sweep is cut."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

DRIVER = r"""
#include "burgers_plan.hpp"
#include <cstdio>
#include <initializer_list>

template <int REM> static int pass(int m)
{
    int slot_of[4] = {-1, -1, -1, -1}, requests = 0, next = m - 1, in_flight = 0, bad = 0;
    sadj::stored_reverse_schedule<4, REM>(
        m,
        [&](int t, int slot) {
            if (t < 0 || t >= m || slot_of[slot] >= 0) ++bad;
            slot_of[slot] = t;
            ++requests;
            ++in_flight;
        },
        [&](int slot) {
            if (slot_of[slot] != next) ++bad;
            if (in_flight != (next + 1 < 4 ? next + 1 : 4)) ++bad;
            slot_of[slot] = -1;
            --next;
            --in_flight;
        });
    if (requests != m || next != -1) ++bad;
    if (bad) std::printf("pass of %d: %d requests, %d wrong\n", m, requests, bad);
    return bad;
}

struct Ops {
    int first = 0, n = 0, m[32];
    int forward(const char *, char *, long, long, int, char *, bool) { return 1; }
    int reverse(const char *, const char *, int, int, int steps, const char *, char *) { m[n++] = steps; return 0; }
    int reverse_first(const char *, const char *, char *) { ++first; return 0; }
};

int main()
{
    int bad = 0;
    for (int m = 1; m <= 64; ++m) bad += m % 4 == 0 ? pass<0>(m) : m % 4 == 1 ? pass<1>(m) : m % 4 == 2 ? pass<2>(m) : pass<3>(m);
    static char lam[2];
    char *const l[2] = {lam, lam + 1};
    for (size_t row : {(size_t)8, (size_t)1 << 27})
        for (long nsteps = 1; nsteps <= 200; ++nsteps) {
            Ops ops;
            if (sadj::plan_burgers_history_reverse(ops, nullptr, row, nsteps, l)) ++bad;
            int sum = 1, longest = 0, shortest = 99;
            for (int i = 0; i < ops.n; ++i) {
                sum += ops.m[i];
                if (ops.m[i] > longest) longest = ops.m[i];
                if (ops.m[i] < shortest) shortest = ops.m[i];
            }
            if (sum != nsteps || ops.first != 1 || longest > sadj::kReverseSteps) ++bad;
            const bool uneven = ops.n > 1 && longest <= sadj::kShortSteps && shortest == 1 && row == 8;
            if (ops.n && !uneven && longest - shortest > 1) { std::printf("%ld steps cut into %d .. %d\n", nsteps, shortest, longest); ++bad; }
        }
    return bad != 0;
}
"""


def test_every_state_is_requested_once_and_in_time(tmp_path):
    src = tmp_path / "driver.cpp"
    src.write_text(DRIVER)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Wno-unknown-pragmas", "-I",
                           os.path.join(ROOT, "paper_1907_02818_amd", "csrc"), str(src), "-o", str(tmp_path / "driver")])
    p = subprocess.run([str(tmp_path / "driver")], stdout=subprocess.PIPE, text=True)
    assert p.returncode == 0, p.stdout
