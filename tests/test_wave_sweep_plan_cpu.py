"""Host-only test of the launch order of sadj_adjoint_wave3d_steps_fused for two and three steps per pass, replayed
with the planner compiled for the host."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

DRIVER = r"""
#include <cstdio>
%s
int main()
{
    for (int most = 2; most <= 3; ++most)
        for (long n = 0; n <= 400; ++n) {
            const WaveSweepPlan p = plan_wave_sweep(n, most);
            if (p.plain) { if (n >= 3) { std::printf("no plan for %%ld\n", n); return 1; } continue; }
            int a = 1, b = 2;
            long steps = 1, launches = 1 + p.body + p.tail_len;
            if (p.body %% 2) { a = 0; b = 3; }
            steps += most * p.body;
            for (int i = 0; i < p.tail_len; ++i) {
                const WaveStepLaunch &l = p.tail[i];
                if (l.a != a || l.b != b || l.steps < 1 || l.steps > most || l.o0 == a || l.o0 == b || l.o0 < 0 || l.o0 > 3) return 2;
                if (l.steps > 1 && (l.o1 == a || l.o1 == b || l.o1 == l.o0 || l.o1 < 0 || l.o1 > 3)) return 3;
                if (l.steps == 1) { a = b; b = l.o0; } else { a = l.o0; b = l.o1; }
                steps += l.steps;
            }
            if (steps != n || a != n %% 3 || b != (n + 1) %% 3) { std::printf("n %%ld most %%d ends wrong\n", n, most); return 4; }
            if (launches > 1 + (n - 1 + most - 1) / most + 3) { std::printf("n %%ld most %%d: %%ld launches\n", n, most, launches); return 5; }
        }
    return 0;
}
"""


def test_sweeps_end_in_the_documented_buffers(tmp_path):
    text = open(os.path.join(ROOT, "paper_1907_02818_amd", "csrc", "api.hip")).read()
    i = text.index("struct WaveStepLaunch")
    j = text.index("// Scratch memory of the entry point that must not allocate")
    src = tmp_path / "driver.cpp"
    src.write_text(DRIVER % re.sub(r"^}  // namespace.*$", "", text[i:j], flags=re.M))
    subprocess.check_call(["g++", "-std=c++17", "-O1", str(src), "-o", str(tmp_path / "driver")])
    p = subprocess.run([str(tmp_path / "driver")], stdout=subprocess.PIPE, text=True)
    assert p.returncode == 0, (p.returncode, p.stdout)
