"""GPU parity of the two-step passes in 64 x 16 tiles, which small grids take (fp64; fp32 grids take tiles of the same size whose
requests run ahead): exact on dyadic data at the edges of those tiles, one and several planes per chunk, NaN where values must not be read."""
import numpy as np
import pytest

import inputs
import oracle
from parity import to_gpu, to_host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sadj():
    import paper_1907_02818_amd as lib
    lib.load()
    return lib


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("shape", [(3, 3, 4), (24, 16, 64), (25, 17, 68), (40, 15, 60), (64, 33, 128), (65, 48, 132), (90, 34, 192), (101, 50, 96)])
def test_small_tiles_are_exact_on_dyadic_data(sadj, shape, dtype):
    """c a multiple of 1/4, adjoints multiples of one: six steps in fp64 and three in fp32 are exact (each step adds
    two bits below the point and at most four above, from three)."""
    import torch
    c = np.clip(np.round(inputs.uniform(3, "c", shape, 0, 1) * 4) / 4, 0.0, 1.0)
    lams = [np.clip(np.round(4 * inputs.uniform(5, k, shape, -1, 1)), -4, 4) for k in ("r_bar", "u_bar", "u_prev_bar")]
    inside = np.zeros(shape, dtype=bool)
    inside[1:-1, 1:-1, 1:-1] = True
    for nsteps in (3,) if dtype == np.float32 else (3, 5, 6):
        want = oracle.wave_adjoint_steps(c, *lams, 1, nsteps)
        g = [to_gpu(x.astype(dtype)) for x in (np.where(inside, lams[0], np.nan), lams[1], lams[2])]
        work = torch.full_like(g[0], float("nan"))
        sadj.sadj_adjoint_wave3d_steps_fused(1, nsteps, to_gpu(np.where(inside, c, np.nan).astype(dtype)), *g, work)
        torch.cuda.synchronize()
        for k in (nsteps % 3, (nsteps + 1) % 3):
            assert np.array_equal(to_host(g[k]).astype(np.float64), want[k]), (nsteps, k)
