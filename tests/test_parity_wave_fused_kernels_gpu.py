"""GPU test that a fused wave sweep has the same bits in the march with its requests ahead and in the tiles of larger grids (option
"wave3d.ahead" 1), on data whose sums round: two and three steps per pass, at the edges of the tiles of both, several cuts."""
import numpy as np
import pytest

import inputs
from parity import to_gpu
from test_parity_wave_pair_ahead_gpu import SHAPES, SHAPES3

pytestmark = pytest.mark.gpu

# tiles whose frame lies in the grid (fp64 64 x 32, fp32 128 x 32 cells) as well; few long rows, beyond the bytes of the other shapes
CORE = [(np.float64, (40, 100, 260)), (np.float32, (40, 100, 520)), (np.float32, (33, 70, 388)), (np.float32, (6, 16, 200000))]


@pytest.fixture
def sadj():
    import paper_1907_02818_amd as lib
    lib.load()
    yield lib
    lib.set_option("wave3d.ahead", 0)
    lib.set_option("wave3d.zchunk", 0)


@pytest.mark.parametrize("dtype,shape", [(d, s) for t in (SHAPES, SHAPES3) for d in t for s in t[d]] + CORE)
def test_same_bits_in_both_kernels(sadj, dtype, shape):
    import torch
    c = to_gpu(inputs.uniform(3, "c", shape, 0.01, 0.1).astype(dtype))
    lams = [to_gpu(inputs.uniform(5, k, shape, -1, 1).astype(dtype)) for k in ("r_bar", "u_bar", "u_prev_bar")]
    for nsteps in (3, 8):
        want = None
        for off, zchunk in ((0, 0), (1, 0), (0, 3), (1, 3), (1, 1000)):
            g = [x.clone() for x in lams]
            sadj.set_option("wave3d.ahead", off)
            sadj.set_option("wave3d.zchunk", zchunk)
            sadj.sadj_adjoint_wave3d_steps_fused(1, nsteps, c, *g, torch.full_like(c, float("nan")))
            got = [g[nsteps % 3], g[(nsteps + 1) % 3]]
            want = want or got
            assert all(torch.isfinite(x).all() for x in got)
            for k, (x, y) in enumerate(zip(got, want)):
                assert torch.equal(x, y), (nsteps, off, zchunk, k, int((x != y).sum()))
