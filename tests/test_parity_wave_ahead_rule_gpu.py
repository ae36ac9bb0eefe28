"""GPU test of the grids that the march with its requests ahead takes beyond those of test_parity_wave_pair_ahead_gpu: fp64 grids of 16 planes
and more in small tiles, and three steps per pass on grids of up to 600 MB (fp32) and 1.2 GB.  The bits are those of the tiles of larger
grids (option "wave3d.ahead" 1) on data whose sums round, and NaN outside I is not read."""
import numpy as np
import pytest

import inputs
from parity import to_gpu

pytestmark = pytest.mark.gpu

GRIDS = [(np.float64, (16, 17, 66)), (np.float64, (33, 32, 224)), (np.float64, (19, 76, 468)), (np.float64, (52, 740, 164)),
         (np.float64, (68, 184, 1012)), (np.float32, (32, 896, 300)), (np.float32, (44, 260, 968)), (np.float32, (560, 652, 44))]


@pytest.fixture
def sadj():
    import paper_1907_02818_amd as lib
    lib.load()
    yield lib
    lib.set_option("wave3d.ahead", 0)


@pytest.mark.parametrize("dtype,shape", GRIDS)
def test_same_bits_in_both_kernels(sadj, dtype, shape):
    import torch
    inside = np.zeros(shape, dtype=bool)
    inside[1:-1, 1:-1, 1:-1] = True
    c, l0 = (np.where(inside, x, np.nan) for x in (inputs.uniform(3, "c", shape, 0.01, 0.1), inputs.uniform(5, "r_bar", shape, -1, 1)))
    c, lams = to_gpu(c.astype(dtype)), [to_gpu(x.astype(dtype)) for x in (l0, inputs.uniform(5, "u_bar", shape, -1, 1), l0 * 0 + 1)]
    lams[2].nan_to_num_(0.0)
    for nsteps in (3, 7):
        want = None
        for off in (1, 0):
            g = [x.clone() for x in lams]
            sadj.set_option("wave3d.ahead", off)
            sadj.sadj_adjoint_wave3d_steps_fused(1, nsteps, c, *g, torch.full_like(c, float("nan")))
            got = [g[nsteps % 3], g[(nsteps + 1) % 3]]
            want = want or got
            assert all(torch.isfinite(x).all() for x in got)
            for x, y in zip(got, want):
                assert torch.equal(x, y), (nsteps, int((x != y).sum()))
