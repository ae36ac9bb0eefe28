"""GPU parity of the three-step passes of sadj_adjoint_wave3d_steps_fused.  Grids as small as these take two
steps per pass by default; z-chunks of 5 planes (fp32: 9) and more make the sweep take three."""
import numpy as np
import pytest

import inputs
import oracle
from parity import TOL, to_gpu, to_host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sadj():
    import paper_1907_02818_amd as lib
    lib.load()
    yield lib
    lib.set_option("wave3d.zchunk", 0)


def _run(sadj, nsteps, zchunk, c, lams):
    import torch
    g = [to_gpu(x) for x in lams]
    work = torch.full_like(g[0], float("nan"))
    sadj.set_option("wave3d.zchunk", zchunk)
    sadj.sadj_adjoint_wave3d_steps_fused(1, nsteps, to_gpu(c), *g, work)
    sadj.set_option("wave3d.zchunk", 0)
    torch.cuda.synchronize()
    return [to_host(t) for t in g]


# tile 64 x 32 (fp32: 128 x 32): edges of tiles, frames that leave the grid, axes without core cells, several chunks with a short last one
SHAPES = [(3, 3, 4), (5, 3, 8), (6, 7, 12), (21, 37, 150), (40, 35, 262), (9, 70, 136), (33, 3, 68), (13, 32, 64), (14, 33, 128), (25, 96, 196), (61, 20, 24)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("zchunk", [5, 7, 100])
def test_three_step_passes_are_exact_on_dyadic_data(sadj, shape, zchunk):
    """c a multiple of 1/4, adjoints small integers: every sum of up to seven steps is exact in fp64, so the
    GPU returns the oracle's numbers bit for bit."""
    c = np.clip(np.round(inputs.uniform(3, "c", shape, 0, 1) * 4) / 4, 0.0, 1.0)
    lams = [np.clip(np.round(4 * inputs.uniform(5, k, shape, -1, 1)), -4, 4) for k in ("r_bar", "u_bar", "u_prev_bar")]
    inside = np.zeros(shape, dtype=bool)
    inside[1:-1, 1:-1, 1:-1] = True
    for nsteps in (4, 5, 6, 7):
        want = oracle.wave_adjoint_steps(c, *lams, 1, nsteps)
        cn, l0 = np.where(inside, c, np.nan), np.where(inside, lams[0], np.nan)     # outside I: never used
        got = _run(sadj, nsteps, zchunk, cn, [l0, lams[1], lams[2]])
        for k in (nsteps % 3, (nsteps + 1) % 3):
            assert np.array_equal(got[k], want[k]), "buffer %d after %d steps: %d cells differ" % (
                k, nsteps, int(np.sum(got[k] != want[k])))


@pytest.mark.parametrize("dtype,zchunk", [(np.float64, 6), (np.float32, 9), (np.float32, 100)])
@pytest.mark.parametrize("shape", [(21, 37, 152), (40, 35, 264), (3, 3, 4), (10, 65, 256)])
def test_three_step_passes_match_the_oracle(sadj, shape, dtype, zchunk):
    """Real-valued inputs within the rounding of the terms: each step adds at most 9 of them, so the relative
    error of a sweep stays below nsteps times the single-step tolerance of the largest value."""
    c = inputs.uniform(1, "c", shape, 0.01, 0.1).astype(dtype)
    lams = [inputs.uniform(2, k, shape, -1, 1).astype(dtype) for k in ("r_bar", "u_bar", "u_prev_bar")]
    for nsteps in (7, 10, 14):
        want = oracle.wave_adjoint_steps(c, *lams, 1, nsteps)
        got = _run(sadj, nsteps, zchunk, c, lams)
        for k in (nsteps % 3, (nsteps + 1) % 3):
            g = got[k].astype(np.float64)
            assert np.isfinite(g).all()
            assert np.max(np.abs(g - want[k])) <= TOL[np.dtype(dtype)] * nsteps * max(np.max(np.abs(want[k])), 1e-300)
