"""GPU tests of the Burgers time loops that take several steps per pass over the data (option
"burgers1d.fuse" 0, the default) against one launch per step (1): the same bits everywhere, at
the edges of the windows a wave owns, for rows of odd length, for passes that meet checkpoints and
for every remainder of the steps a pass can take."""
import numpy as np
import pytest

import inputs
from parity import to_gpu, to_host

pytestmark = pytest.mark.gpu

BC, BD = 0.1, 0.05
# windows own 96 cells in short arrays; from 1024 windows of 224 (fp64) / 480 (fp32) cells on they own
# that many
SIZES = [3, 4, 95, 96, 97, 110, 112, 113, 192, 1001]
WIDE = {np.float64: [229375, 229376, 229600, 230017], np.float32: [491519, 491520, 492000, 492483]}


@pytest.fixture(scope="module")
def sadj():
    import paper_1907_02818_amd as lib
    lib.load()
    yield lib
    lib.set_option("burgers1d.fuse", 0)


def _both(sadj, fn):
    """fn() with one launch per step, then with several steps per pass."""
    import torch
    out = []
    for fuse in (1, 0):
        sadj.set_option("burgers1d.fuse", fuse)
        r = fn()
        torch.cuda.synchronize()
        out.append([to_host(t) for t in r])
    sadj.set_option("burgers1d.fuse", 0)
    return out


def _lam(n, dtype):
    lam0 = inputs.uniform(n, "r_bar", (n,), -1, 1).astype(dtype)
    lam0[0] = lam0[-1] = np.nan                       # outside I: never used
    return lam0, inputs.uniform(n, "u_bar", (n,), -1, 1).astype(dtype)


def _history(sadj, n, nsteps, dtype):
    u0 = inputs.burgers_inputs(n, seed=n, dtype=dtype)["u"]
    st = np.full((nsteps + 1, n), np.nan, dtype=dtype)
    st[0] = u0
    for t in range(1, nsteps + 1):                    # boundary data of its own in every row
        st[t, 0], st[t, -1] = 0.3 * np.sin(t), -0.2 * np.cos(t)
    lam0, lam1 = _lam(n, dtype)

    def go():
        g, a, b = to_gpu(st), to_gpu(lam0), to_gpu(lam1)
        sadj.sadj_primal_burgers1d_steps(BC, BD, nsteps, g)
        sadj.sadj_adjoint_burgers1d_steps(BC, BD, nsteps, nsteps, g, a, b)
        return g, (a, b)[nsteps % 2]

    want, got = _both(sadj, go)
    for w, g in zip(want, got):
        assert np.isfinite(w).all() and np.array_equal(w, g)


def _ckpt(sadj, n, nsteps, every, dtype):
    u0 = inputs.burgers_inputs(n, seed=n + every, dtype=dtype)["u"]
    ck = np.full((nsteps // every + 1, n), np.nan, dtype=dtype)
    ck[0] = u0
    lam0, lam1 = _lam(n, dtype)

    def go():
        g, a, b = to_gpu(ck), to_gpu(lam0), to_gpu(lam1)
        work, fin = to_gpu(np.full((2, n), np.nan, dtype=dtype)), to_gpu(np.full(n, np.nan, dtype=dtype))
        sadj.sadj_primal_burgers1d_ckpt(BC, BD, nsteps, every, g, work, fin)
        wk = to_gpu(np.full((every - 1) * n, np.nan, dtype=dtype)) if every > 1 else None
        sadj.sadj_adjoint_burgers1d_ckpt(BC, BD, nsteps, every, g, wk, a, b)
        return g, fin, (a, b)[nsteps % 2]

    want, got = _both(sadj, go)
    for w, g in zip(want, got):
        assert np.isfinite(w).all() and np.array_equal(w, g)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("n", SIZES)
def test_stored_states_short_arrays(sadj, n, dtype):
    for nsteps in (1, 2, 15, 16, 17, 18, 33):
        _history(sadj, n, nsteps, dtype)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("k", range(4))
def test_stored_states_wide_windows(sadj, k, dtype):
    for nsteps in (5, 18):
        _history(sadj, WIDE[dtype][k], nsteps, dtype)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("n", SIZES)
def test_checkpoints_short_arrays(sadj, n, dtype):
    for nsteps, every in [(1, 2), (3, 2), (7, 3), (9, 4), (16, 8), (18, 9), (40, 16), (41, 19), (6, 7), (50, 40)]:
        _ckpt(sadj, n, nsteps, every, dtype)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("k", range(4))
def test_checkpoints_wide_windows(sadj, k, dtype):
    for nsteps, every in [(17, 8), (21, 11), (9, 3)]:
        _ckpt(sadj, WIDE[dtype][k], nsteps, every, dtype)
