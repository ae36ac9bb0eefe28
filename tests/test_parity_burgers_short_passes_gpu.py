"""GPU test of the Burgers reverse sweep over stored states for every length of a pass and of its remainders, at
the edges of the windows of short passes (112 cells, from 229376 fp64 / 491520 fp32 cells on 240 / 496) and for
rows that are not 16-byte aligned: the same bits as one launch per step."""
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
    lib.set_option("burgers1d.fuse", 0)


def _same_bits(sadj, n, nsteps, dtype):
    import torch
    states = to_gpu(inputs.uniform(n + nsteps, "u", (nsteps, n), -0.5, 0.5).astype(dtype))
    states = torch.cat([states, states[:1]])
    lam = [inputs.uniform(n, k, (n,), -1, 1).astype(dtype) for k in ("r_bar", "u_bar")]
    lam[0][0] = lam[0][-1] = np.nan                       # outside I: never used
    out = []
    for fuse in (1, 0):
        sadj.set_option("burgers1d.fuse", fuse)
        g = [to_gpu(x) for x in lam]
        sadj.sadj_adjoint_burgers1d_steps(0.1, 0.05, nsteps, nsteps, states, *g)
        torch.cuda.synchronize()
        out.append(to_host(g[nsteps % 2]))
    sadj.set_option("burgers1d.fuse", 0)
    assert np.isfinite(out[0]).all() and np.array_equal(out[0], out[1]), (n, nsteps)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("n", [3, 8, 97, 103, 104, 105, 111, 112, 113, 120, 224, 225, 1024])
def test_short_arrays(sadj, n, dtype):
    for nsteps in list(range(2, 17)) + [22, 30]:
        _same_bits(sadj, n, nsteps, dtype)


@pytest.mark.parametrize("dtype,n", [(np.float64, 229440), (np.float64, 229441), (np.float64, 229681), (np.float32, 492032),
                                     (np.float32, 492033), (np.float32, 492527)])
def test_wide_windows(sadj, n, dtype):
    for nsteps in (2, 3, 4, 5, 6, 8, 9, 11, 14, 16):
        _same_bits(sadj, n, nsteps, dtype)
