"""GPU tests of the Burgers step, its adjoint and their time loops where states are not finite: NaN and infinities beside cells of
either sign and beside zeros propagate as in the formula, whose products with 0 give NaN; the loops that take several steps per
pass do so as one launch per step does, also where finite states overflow on the way."""
import numpy as np
import pytest

import inputs
import oracle
from parity import assert_close, to_gpu, to_host

pytestmark = pytest.mark.gpu

BC, BD = 0.1, 0.05


@pytest.fixture(scope="module")
def sadj():
    import paper_1907_02818_amd as lib
    lib.load()
    yield lib
    lib.set_option("burgers1d.fuse", 0)


def _state(n, dtype, every=23):
    """Uniform values with a NaN or an infinity every few cells, zeros of both signs among their neighbours."""
    u = inputs.uniform(n, "u", (n,), -1, 1).astype(dtype)
    at = np.arange(1, n - 1, every)
    u[at] = np.array([np.nan, np.inf, -np.inf], dtype)[np.arange(at.size) % 3]
    u[at[2::5] + 1] = 0.0
    u[at[3::5] - 1] = -0.0
    return u


def _same_kind(got, want):
    return (np.isnan(got) == np.isnan(want)) & (np.isinf(got) == np.isinf(want)) & (~np.isinf(want) | (np.sign(got) == np.sign(want)))


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("n", [3, 65, 300, 4097])
def test_one_step_and_its_adjoint_propagate_as_the_formula(sadj, n, dtype):
    u = _state(n, dtype, every=23 if n > 3 else 1)
    r_bar, u_bar = (inputs.uniform(n, k, (n,), -1, 1).astype(dtype) for k in ("r_bar", "u_bar"))
    with np.errstate(all="ignore"):
        want, (want_b, scale) = oracle.burgers_primal(u, BC, BD), oracle.burgers_adjoint(u, r_bar, u_bar, BC, BD, want_scale=True)
        r, b = to_gpu(np.zeros_like(u)), to_gpu(u_bar)
        sadj.sadj_primal_burgers1d(BC, BD, to_gpu(u), r)
        sadj.sadj_adjoint_burgers1d(BC, BD, to_gpu(u), to_gpu(r_bar), b)
        r, b = to_host(r), to_host(b)
        assert n == 3 or (np.isnan(want).any() and np.isinf(want).any() and np.isnan(want_b).any() and np.isinf(want_b).any())
        assert _same_kind(r[1:-1], want[1:-1]).all(), np.flatnonzero(~_same_kind(r, want))
        assert _same_kind(b, want_b).all(), np.flatnonzero(~_same_kind(b, want_b))
        ok = np.isfinite(want_b)
        if ok.any():
            assert_close(b[ok], want_b[ok], scale[ok] + np.abs(u_bar[ok]), dtype, "adjoint n=%d" % n)


def _loops(sadj, u0, nsteps, every):
    n = u0.size
    lam0, lam1 = (inputs.uniform(n, k, (n,), -1, 1).astype(u0.dtype) for k in ("r_bar", "u_bar"))
    states = np.stack([u0] + [np.zeros_like(u0)] * nsteps)
    if not np.isfinite(u0[[0, -1]]).all():             # end cells are given in every row
        states[3::4, 0], states[1::5, -1] = -np.inf, np.nan
    states = to_gpu(states)
    g = [to_gpu(lam0), to_gpu(lam1)]
    sadj.sadj_primal_burgers1d_steps(BC, BD, nsteps, states)
    sadj.sadj_adjoint_burgers1d_steps(BC, BD, nsteps, nsteps, states, *g)
    ck = to_gpu(np.stack([u0] + [np.zeros_like(u0)] * (nsteps // every)))
    work, fin, h = to_gpu(np.zeros((max(2, every - 1), n), u0.dtype)), to_gpu(np.zeros_like(u0)), [to_gpu(lam0), to_gpu(lam1)]
    sadj.sadj_primal_burgers1d_ckpt(BC, BD, nsteps, every, ck, work, fin)
    sadj.sadj_adjoint_burgers1d_ckpt(BC, BD, nsteps, every, ck, work, *h)
    return [to_host(t) for t in (states, g[nsteps % 2], ck, fin, h[nsteps % 2])]


@pytest.mark.parametrize("n,dtype", [(300, np.float64), (300, np.float32), (1021, np.float64), (1021, np.float32), (229633, np.float64),
                                     (492064, np.float32)])
def test_loops_propagate_as_one_launch_per_step(sadj, n, dtype):
    few = _state(n, dtype, every=211)
    blown_up = inputs.uniform(n, "u", (n,), -1, 1).astype(dtype) * dtype(1e100 if dtype == np.float64 else 1e12)
    blown_up[n // 2:] = few[n // 2:]                   # some windows overflow, others meet what is not finite, or neither
    few[n // 2:] = inputs.uniform(n, "u", (n,), -1, 1).astype(dtype)[n // 2:]
    ends = inputs.uniform(n, "u", (n,), -1, 1).astype(dtype)
    ends[0], ends[-1] = np.inf, -np.inf
    for u0 in (few, blown_up, ends):
        for nsteps, every in ((1, 2), (5, 3), (17, 16), (34, 16), (13, 12), (18, 17), (9, 2)):
            out = []
            for fuse in (1, 0):
                sadj.set_option("burgers1d.fuse", fuse)
                out.append(_loops(sadj, u0, nsteps, every))
            sadj.set_option("burgers1d.fuse", 0)
            assert not np.isfinite(out[0][0]).all() and np.isfinite(out[0][0][-1]).any()
            for k, (x, y) in enumerate(zip(*out)):
                assert np.array_equal(x, y, equal_nan=True), (nsteps, every, k)
