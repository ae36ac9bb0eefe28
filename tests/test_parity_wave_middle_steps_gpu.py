"""GPU test of the middle steps of a wave time loop (sadj_adjoint_wave3d_steps from its third step on:
the start value of u_bar is read as the negated r_bar of the step before instead of being written and
read back): the same bits as single calls on zeroed buffers, for tile edges, empty cores, rows that
are no whole vectors, several z-chunks, and with NaN where values must not be read."""
import numpy as np
import pytest

import inputs
from parity import to_gpu, to_host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sadj():
    import paper_1907_02818_amd as lib
    lib.load()
    yield lib
    lib.set_option("wave3d.zchunk", 0)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("radius,shape", [(1, (3, 3, 3)), (1, (20, 33, 66)), (1, (9, 40, 131)), (2, (5, 5, 8)), (2, (40, 31, 130)),
                                          (3, (13, 34, 65)), (4, (9, 9, 9)), (4, (30, 34, 132)), (4, (41, 20, 250))])
def test_middle_steps_equal_single_calls_bitwise(sadj, radius, shape, dtype):
    import torch
    c = inputs.uniform(1, "c", shape, 0.01, 0.1).astype(dtype)
    inside = np.zeros(shape, dtype=bool)
    inside[tuple(slice(radius, n - radius) for n in shape)] = True
    c[~inside] = np.nan                                    # never read outside I
    lams = [inputs.uniform(7, k, shape, -1, 1).astype(dtype) for k in ("r_bar", "u_bar", "u_prev_bar")]
    cg = to_gpu(c)
    for zchunk in (0, 3):
        sadj.set_option("wave3d.zchunk", zchunk)
        for nsteps in (2, 3, 4, 5):
            g = [to_gpu(x) for x in lams]
            sadj.sadj_adjoint_wave3d_steps(radius, nsteps, cg, *g)
            h = [to_gpu(x) for x in lams]
            for s in range(nsteps):
                a, b, p = h[s % 3], h[(s + 1) % 3], h[(s + 2) % 3]
                if s > 0:
                    p.zero_()
                sadj.sadj_adjoint_wave3d(radius, cg, a, b, p)
            torch.cuda.synchronize()
            for k in (nsteps % 3, (nsteps + 1) % 3):
                want = to_host(h[k])
                assert np.isfinite(want).all()
                assert np.array_equal(to_host(g[k]), want), (zchunk, nsteps, k)
    sadj.set_option("wave3d.zchunk", 0)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("radius,shape", [(1, (30, 36, 140)), (2, (40, 37, 132)), (2, (31, 70, 260)), (3, (45, 40, 136)), (3, (33, 71, 259)),
                                          (4, (50, 44, 140)), (4, (40, 75, 264))])
def test_middle_steps_of_long_marches(sadj, radius, shape, dtype):
    """Chunks much longer than R + 2 planes, where the fp32 kernels run their phase without conditions on the plane, in
    tiles inside the grid and at its edge; the same bits as single calls, and as any other cut."""
    import torch
    c = to_gpu(inputs.uniform(1, "c", shape, 0.01, 0.1).astype(dtype))
    lams = [to_gpu(inputs.uniform(7, k, shape, -1, 1).astype(dtype)) for k in ("r_bar", "u_bar", "u_prev_bar")]
    nsteps, want = 5, [x.clone() for x in lams]
    for s in range(nsteps):
        a, b, p = want[s % 3], want[(s + 1) % 3], want[(s + 2) % 3]
        if s > 0:
            p.zero_()
        sadj.sadj_adjoint_wave3d(radius, c, a, b, p)
    for zchunk in (0, 17, 1000):
        sadj.set_option("wave3d.zchunk", zchunk)
        g = [x.clone() for x in lams]
        sadj.sadj_adjoint_wave3d_steps(radius, nsteps, c, *g)
        sadj.set_option("wave3d.zchunk", 0)
        for k in (nsteps % 3, (nsteps + 1) % 3):
            assert torch.isfinite(want[k]).all() and torch.equal(g[k], want[k]), (zchunk, k)
