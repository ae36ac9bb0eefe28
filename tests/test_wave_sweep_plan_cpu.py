"""Host-only test of the launch order of sadj_adjoint_wave3d_steps_fused for two and three steps per pass, replayed
with the planner compiled for the host, and of the diagnostic that shows it."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

DRIVER = r"""
#include "wave_sweep_plan.hpp"
#include <cstdio>
using namespace sadj;
int main()
{
    for (int most = 2; most <= 3; ++most)
        for (long n = 0; n <= 400; ++n) {
            const WaveSweepPlan p = plan_wave_sweep(n, most);
            if (p.plain) { if (n >= 3) { std::printf("no plan for %ld\n", n); return 1; } continue; }
            int a = 1, b = 2;
            long steps = 1, launches = 1 + p.body + p.tail_len;
            if (p.body % 2) { a = 0; b = 3; }
            steps += most * p.body;
            for (int i = 0; i < p.tail_len; ++i) {
                const WaveStepLaunch &l = p.tail[i];
                if (l.a != a || l.b != b || l.steps < 1 || l.steps > most || l.o0 == a || l.o0 == b || l.o0 < 0 || l.o0 > 3) return 2;
                if (l.steps > 1 && (l.o1 == a || l.o1 == b || l.o1 == l.o0 || l.o1 < 0 || l.o1 > 3)) return 3;
                if (l.steps == 1) { a = b; b = l.o0; } else { a = l.o0; b = l.o1; }
                steps += l.steps;
            }
            if (steps != n || a != n % 3 || b != (n + 1) % 3) { std::printf("n %ld most %d ends wrong\n", n, most); return 4; }
            if (launches > 1 + (n - 1 + most - 1) / most + 3) { std::printf("n %ld most %d: %ld launches\n", n, most, launches); return 5; }
        }
    return 0;
}
"""


def test_sweeps_end_in_the_documented_buffers(tmp_path):
    src = tmp_path / "driver.cpp"
    src.write_text(DRIVER)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_1907_02818_amd", "csrc"), str(src), "-o", str(tmp_path / "driver")])
    p = subprocess.run([str(tmp_path / "driver")], stdout=subprocess.PIPE, text=True)
    assert p.returncode == 0, (p.returncode, p.stdout)


@pytest.mark.parametrize("dtype_code,shape,steps", [(1, (512, 512, 512), 3), (1, (128, 128, 128), 3), (0, (192, 192, 192), 3),
                                                    (1, (24, 24, 24), 2), (0, (96, 130, 164), 2)])
def test_the_diagnostic_shows_the_launches_of_this_grid(dtype_code, shape, steps):
    """Every launch writes buffers that it does not read, the steps add up and the results end where the header
    says, for the number of steps per pass that the grid takes."""
    torch = pytest.importorskip("torch")
    if torch.cuda.is_available():
        pytest.skip("plans depend on the device's compute units; this test counts on the default")
    import paper_1907_02818_amd as lib
    nz, ny, nx = shape
    for n in (3, 4, 7, 25, 26, 27, 100):
        body, body_steps, tail = lib.sadj_describe_wave3d_sweep_launches(dtype_code, 1, nx, ny, nz, n)
        assert body_steps == steps and body >= 0
        a, b = (1, 2) if body % 2 == 0 else (0, 3)
        total = 1 + steps * body
        for k, la, lb, o0, o1 in tail:
            assert (la, lb) == (a, b) and 1 <= k <= steps and len({la, lb, o0} | ({o1} if k > 1 else set())) == (4 if k > 1 else 3)
            a, b = (o0, o1) if k > 1 else (lb, o0)
            total += k
        assert total == n and (a, b) == (n % 3, (n + 1) % 3)


def test_the_diagnostic_shows_where_single_steps_run():
    import paper_1907_02818_amd as lib
    assert lib.sadj_describe_wave3d_sweep_launches(1, 1, 512, 512, 512, 2) == (-1, 1, [])
    assert lib.sadj_describe_wave3d_sweep_launches(1, 1, 511, 512, 512, 25) == (-1, 1, [])
    assert lib.sadj_describe_wave3d_sweep_launches(0, 1, 510, 512, 512, 25) == (-1, 1, [])
    assert lib.sadj_describe_wave3d_sweep_launches(1, 4, 512, 512, 512, 25) == (-1, 1, [])
    lib.set_option("wave3d.fuse", 1)
    try:
        assert lib.sadj_describe_wave3d_sweep_launches(1, 1, 512, 512, 512, 25) == (-1, 1, [])
    finally:
        lib.set_option("wave3d.fuse", 0)
    for bad in ((1, 5, 64, 64, 64, 4), (1, 1, 2, 64, 64, 4), (1, 1, 64, 64, 64, -1), (2, 1, 64, 64, 64, 4)):
        with pytest.raises(lib.SadjError):
            lib.sadj_describe_wave3d_sweep_launches(*bad)


def test_options_that_move_work_do_not_change_the_steps_of_a_pass():
    """Two and three steps per pass round differently, and the header promises that these options change no bit."""
    import paper_1907_02818_amd as lib
    grids = [(1, s) for s in ((207, 35, 136), (136, 35, 208), (81, 68, 260), (96, 100, 128), (64, 64, 64), (150, 150, 150), (512, 512, 512))]
    grids += [(0, s) for s in ((96, 130, 164), (197, 68, 260), (160, 180, 200), (64, 64, 64), (512, 512, 512))]
    ask = lambda d, s: lib.sadj_describe_wave3d_sweep_launches(d, 1, s[2], s[1], s[0], 25)   # noqa: E731
    want = [ask(d, s) for d, s in grids]
    for name, values in (("wave3d.zchunk", (1, 5, 9, 100)), ("wave3d.split", (1,)), ("wave3d.ldspad", (-1, 4096)), ("wave3d.xcdmap", (2, 3)),
                         ("wave3d.band", (1, 8))):
        for v in values:
            lib.set_option(name, v)
            try:
                assert [ask(d, s) for d, s in grids] == want, (name, v)
            finally:
                lib.set_option(name, 0)
