"""GPU parity of the two- and three-step passes that request their planes ahead (64 x 16 cells; two steps: fp32 up to 230 MB in five
arrays, fp64 where the grid takes no small tiles or from 30 MB; three steps up to 260 and 300 MB; more grids in
test_parity_wave_ahead_rule_gpu): exact on dyadic data for chunks of one plane to the whole depth, at the edges of tiles and of
the range, NaN where values must not be read."""
import numpy as np
import pytest

import inputs
import oracle
from parity import to_gpu, to_host
from test_parity_wave_triple_gpu import _largest_sum

pytestmark = pytest.mark.gpu

SHAPES = {np.float64: [(97, 65, 132), (300, 50, 62), (46, 130, 128), (3, 500, 512), (8, 301, 400), (75, 247, 310)],
          np.float32: [(3, 3, 4), (5, 17, 68), (24, 33, 64), (197, 68, 260), (8, 1000, 1024), (3, 16, 132), (40, 500, 568)]}


@pytest.fixture(scope="module")
def sadj():
    import paper_1907_02818_amd as lib
    lib.load()
    yield lib
    lib.set_option("wave3d.zchunk", 0)


@pytest.mark.parametrize("dtype,shape", [(d, s) for d in SHAPES for s in SHAPES[d]])
def test_passes_that_request_ahead_are_exact_on_dyadic_data(sadj, dtype, shape):
    """c a multiple of 1/4, adjoints whole numbers up to 4: three steps, one alone and two in one pass, are exact in both types."""
    import torch
    c = np.clip(np.round(inputs.uniform(3, "c", shape, 0, 1) * 4) / 4, 0.0, 1.0)
    lams = [np.clip(np.round(4 * inputs.uniform(5, k, shape, -1, 1)), -4, 4) for k in ("r_bar", "u_bar", "u_prev_bar")]
    inside = np.zeros(shape, dtype=bool)
    inside[1:-1, 1:-1, 1:-1] = True
    want = oracle.wave_adjoint_steps(c, *lams, 1, 3)
    cn, l0 = to_gpu(np.where(inside, c, np.nan).astype(dtype)), np.where(inside, lams[0], np.nan).astype(dtype)
    for zchunk in (0, 1, 2, 3, 7, 1000):
        g = [to_gpu(x.astype(dtype)) for x in (l0, lams[1], lams[2])]
        work = torch.full_like(g[0], float("nan"))
        sadj.set_option("wave3d.zchunk", zchunk)
        sadj.sadj_adjoint_wave3d_steps_fused(1, 3, cn, *g, work)
        sadj.set_option("wave3d.zchunk", 0)
        for k in (0, 1):
            assert np.array_equal(to_host(g[k]).astype(np.float64), want[k]), (zchunk, k)


# grids of three steps per pass: tile edges, a frame that leaves the grid on all sides, thin grids that march few planes beyond the
# wide tiles' and stay there, the largest of the range
SHAPES3 = {np.float64: [(897, 17, 64), (900, 17, 66), (379, 33, 128), (97, 65, 256), (81, 68, 260), (4, 1000, 1026), (100, 240, 310)],
           np.float32: [(897, 33, 64), (449, 37, 152), (197, 68, 260), (8, 1000, 1024), (66, 400, 480)]}


@pytest.mark.parametrize("dtype,shape", [(d, s) for d in SHAPES3 for s in SHAPES3[d]])
def test_three_step_passes_that_request_ahead_are_exact_on_dyadic_data(sadj, dtype, shape):
    """As above over seven steps; fp32: whole numbers, c 0 or 1, so few of them that no sum reaches 2^24."""
    import torch
    steps = 7
    nz, ny, nx = shape
    assert sadj.sadj_describe_wave3d_sweep_launches(1 if dtype == np.float64 else 0, 1, nx, ny, nz, steps)[1] == 3
    c = inputs.uniform(3, "c", shape, 0, 1)
    c = np.clip(np.round(c * 4) / 4, 0.0, 1.0) if dtype == np.float64 else (c < 0.04).astype(np.float64)
    top = 4 if dtype == np.float64 else 0.8
    lams = [np.clip(np.round(top * inputs.uniform(5, k, shape, -1, 1)), -4, 4) for k in ("r_bar", "u_bar", "u_prev_bar")]
    assert dtype == np.float64 or _largest_sum(c, lams, steps) < 2 ** 24
    inside = np.zeros(shape, dtype=bool)
    inside[1:-1, 1:-1, 1:-1] = True
    want = oracle.wave_adjoint_steps(c, *lams, 1, steps)
    cn, l0 = to_gpu(np.where(inside, c, np.nan).astype(dtype)), np.where(inside, lams[0], np.nan).astype(dtype)
    for zchunk in (0, 1, 2, 3, 7, 1000):
        g = [to_gpu(x.astype(dtype)) for x in (l0, lams[1], lams[2])]
        work = torch.full_like(g[0], float("nan"))
        sadj.set_option("wave3d.zchunk", zchunk)
        sadj.sadj_adjoint_wave3d_steps_fused(1, steps, cn, *g, work)
        sadj.set_option("wave3d.zchunk", 0)
        for k in (steps % 3, (steps + 1) % 3):
            assert np.array_equal(to_host(g[k]).astype(np.float64), want[k]), (zchunk, k)
