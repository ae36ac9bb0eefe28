"""CPU test of the tile shape that the 3-D wave primal takes (csrc/shape_rules.hpp): a shape that moves four cells
per lane only where rows and arrays are whole vectors of four, since it would fall back to one cell
per lane elsewhere."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

DRIVER = r"""
#include "shape_rules.hpp"
#include <cstdio>
using sadj::primal_shape;
#define NEED(c) do { if (!(c)) { std::printf("%s\n", #c); bad = 1; } } while (0)
int main()
{
    int bad = 0;
    NEED(primal_shape(4, 1, 500, 0x1000) == 11);
    for (int nx : {502, 506, 510, 1010, 1018, 1022}) NEED(primal_shape(4, 1, nx, 0x1000) == 10);
    for (int nx : {500, 508, 1000, 1020}) NEED(primal_shape(4, 1, nx, 0x1008) == 10);
    NEED(primal_shape(4, 1, 512, 0x1000) == 8 && primal_shape(4, 1, 100, 0x1000) == 8);
    NEED(primal_shape(8, 1, 500, 0x1000) == 10 && primal_shape(8, 1, 512, 0x1000) == 3);
    NEED(primal_shape(8, 4, 500, 0x1000) == 5 && primal_shape(4, 4, 500, 0x1000) == 5 && primal_shape(4, 4, 512, 0x1000) == 8);
    for (int nx = 3; nx < 3000; ++nx)
        for (uintptr_t at : {(uintptr_t)0x1000, (uintptr_t)0x1004, (uintptr_t)0x1008})
            if (primal_shape(4, 1, nx, at) == 11) NEED(nx % 4 == 0 && at % 16 == 0);
    return bad;
}
"""


def test_wide_tiles_only_where_their_vectors_are_whole(tmp_path):
    src = tmp_path / "driver.cpp"
    src.write_text(DRIVER.replace("#include <cstdio>", "#include <cstdio>\n#include <initializer_list>"))
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Wno-unused-function", "-I",
                           os.path.join(ROOT, "paper_1907_02818_amd", "csrc"), str(src), "-o", str(tmp_path / "driver")])
    p = subprocess.run([str(tmp_path / "driver")], stdout=subprocess.PIPE, text=True)
    assert p.returncode == 0, p.stdout
