"""GPU tests of the Burgers reverse sweep where a state is exactly zero over a stretch (both one-sided differences count, for
either sign of the zero), and of passes that recompute up to 8, 12 and 16 states at the edges of their windows (96, 80, 64 own
cells in short arrays; 224, 208, 192 in fp64 and 480, 464, 448 in fp32 from 229376 and 491520 cells on): the same bits as one
launch per step, and the oracle's values."""
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


def _both(sadj, fn):
    out = []
    for fuse in (1, 0):
        sadj.set_option("burgers1d.fuse", fuse)
        out.append([to_host(t) for t in fn()])
    sadj.set_option("burgers1d.fuse", 0)
    return out


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("n", [65, 300, 1021])
def test_states_that_are_zero_over_a_stretch(sadj, n, dtype):
    u = inputs.uniform(n, "u", (n,), -1, 1).astype(dtype)
    u[n // 4: n // 2] = 0.0
    u[n // 3: n // 2: 3] = -0.0
    r_bar, u_bar = (inputs.uniform(n, k, (n,), -1, 1).astype(dtype) for k in ("r_bar", "u_bar"))
    got = to_gpu(u_bar)
    sadj.sadj_adjoint_burgers1d(BC, BD, to_gpu(u), to_gpu(r_bar), got)
    want, scale = oracle.burgers_adjoint(u, r_bar, u_bar, BC, BD, want_scale=True)
    assert_close(to_host(got), want, scale + np.abs(u_bar), dtype, "zero states n=%d" % n)
    states = to_gpu(np.stack([u] * 6))

    def sweep():
        lam = [to_gpu(r_bar), to_gpu(u_bar)]
        sadj.sadj_adjoint_burgers1d_steps(BC, BD, 5, 5, states, *lam)
        return [lam[5 % 2]]

    single, fused = _both(sadj, sweep)
    assert np.isfinite(single[0]).all() and np.array_equal(single[0], fused[0])


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("n", [3, 63, 65, 80, 81, 129, 193, 961, 229632, 229633, 492064])
def test_passes_of_every_length(sadj, n, dtype):
    u0 = inputs.burgers_inputs(n, seed=n, dtype=dtype)["u"]
    u0[n // 2: n // 2 + 5] = 0
    lam0 = inputs.uniform(n, "r_bar", (n,), -1, 1).astype(dtype)
    lam1 = inputs.uniform(n, "u_bar", (n,), -1, 1).astype(dtype)
    for nsteps, every in ((34, 16), (26, 12), (31, 15), (29, 5), (18, 17), (40, 40), (16, 3), (15, 14)):
        def go():
            ck = to_gpu(np.stack([u0] + [np.zeros_like(u0)] * (nsteps // every)))
            work, fin, g = to_gpu(np.zeros((max(2, every - 1), n), dtype)), to_gpu(np.zeros_like(u0)), [to_gpu(lam0), to_gpu(lam1)]
            sadj.sadj_primal_burgers1d_ckpt(BC, BD, nsteps, every, ck, work, fin)
            sadj.sadj_adjoint_burgers1d_ckpt(BC, BD, nsteps, every, ck, work, *g)
            return [ck, fin, g[nsteps % 2]]

        single, fused = _both(sadj, go)
        assert all(np.isfinite(x).all() and np.array_equal(x, y) for x, y in zip(single, fused)), (nsteps, every)


@pytest.mark.parametrize("fuse", [0, 1])
def test_single_precision_roundings_do_not_add_up_to_one_side(sadj, fuse):
    """128 reverse steps over states that are given, another one for each step, against the same in double with C and D as fp32 holds
    them.  A step's roundings are 3.3e-8 of lam; independent from step to step they add up to at most sqrt(128) of that, 3.7e-7
    (bound 6e-7).  1 - 2D rounded by itself is off the same way in every cell and step, which adds up to 3e-6."""
    n, nsteps = 4001, 128
    states = inputs.uniform(1, "u", (nsteps + 1, n), -1, 1).astype(np.float32)
    lam0 = inputs.uniform(n, "r_bar", (n,), -1, 1).astype(np.float32)
    c, d = float(np.float32(BC)), float(np.float32(BD))
    want = lam0.astype(np.float64)
    for k in range(nsteps - 1, -1, -1):
        u = states[k].astype(np.float64)
        um, u0, up = u[:-2], u[1:-1], u[2:]
        slope = np.abs(u0) + (u0 >= 0) * (u0 - um) + (u0 <= 0) * (up - u0)
        r, want = want[1:-1], np.zeros(n)
        want[:-2] += (c * np.maximum(u0, 0) + d) * r
        want[2:] += (-c * np.minimum(u0, 0) + d) * r
        want[1:-1] += (1 - 2 * d - c * slope) * r
    g, lam = to_gpu(states), [to_gpu(lam0), to_gpu(np.zeros_like(lam0))]
    sadj.set_option("burgers1d.fuse", fuse)
    sadj.sadj_adjoint_burgers1d_steps(BC, BD, nsteps, nsteps, g, *lam)
    sadj.set_option("burgers1d.fuse", 0)
    got = to_host(lam[nsteps % 2]).astype(np.float64)
    assert np.linalg.norm(got[1:-1] - want[1:-1]) < 6e-7 * np.linalg.norm(want[1:-1])


def _formula(u, r_bar, c, d):
    """The step and its adjoint as the formula stands, in the type of the arguments."""
    um, u0, up, r = u[:-2], u[1:-1], u[2:], r_bar[1:-1]
    zero = u.dtype.type(0)
    pos, neg = np.maximum(u0, zero), np.minimum(u0, zero)
    step = u0 - c * (pos * (u0 - um) + neg * (up - u0)) + d * (um - 2 * u0 + up)
    adjoint = np.zeros_like(r_bar)
    adjoint[:-2] += (c * pos + d) * r
    adjoint[2:] += (-c * neg + d) * r
    adjoint[1:-1] += (1 - 2 * d - c * ((u0 >= 0) * (u0 - um) + pos + (u0 <= 0) * (up - u0) - neg)) * r
    return step, adjoint


@pytest.mark.parametrize("dtype,wide", [(np.float64, np.longdouble), (np.float32, np.float64)])
def test_one_step_is_no_further_off_than_the_formula_as_it_stands(sadj, dtype, wide):
    """Against wider arithmetic with the same C and D (2-norm): the step 0.71, the adjoint 0.60 to 0.75 of the formula's own error in this type."""
    if np.finfo(wide).eps >= np.finfo(dtype).eps:
        pytest.skip("no wider type here")
    n = 20001
    u = inputs.burgers_inputs(n, seed=2, dtype=dtype)["u"]
    r_bar = inputs.uniform(n, "r_bar", (n,), -1, 1).astype(dtype)
    c, d = dtype(BC), dtype(BD)
    want, plain = _formula(u.astype(wide), r_bar.astype(wide), wide(c), wide(d)), _formula(u, r_bar, c, d)
    r, u_bar = to_gpu(np.zeros_like(u)), to_gpu(np.zeros_like(u))
    sadj.sadj_primal_burgers1d(BC, BD, to_gpu(u), r)
    sadj.sadj_adjoint_burgers1d(BC, BD, to_gpu(u), to_gpu(r_bar), u_bar)
    for got, w, p in zip((to_host(r)[1:-1], to_host(u_bar)), want, plain):
        assert np.linalg.norm(got.astype(wide) - w) <= np.linalg.norm(p.astype(wide) - w)
