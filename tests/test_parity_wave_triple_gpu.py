"""GPU parity of the three-step passes of sadj_adjoint_wave3d_steps_fused, on grids that take three steps per pass and
for several cuts along z."""
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
    nz, ny, nx = c.shape
    g = [to_gpu(x) for x in lams]
    work = torch.full_like(g[0], float("nan"))
    sadj.set_option("wave3d.zchunk", zchunk)
    body, steps, tail = sadj.sadj_describe_wave3d_sweep_launches(1 if c.dtype == np.float64 else 0, 1, nx, ny, nz, nsteps)
    assert steps == 3 and body + sum(t[0] == 3 for t in tail) > 0, "the three-step kernel does not run here"
    sadj.sadj_adjoint_wave3d_steps_fused(1, nsteps, to_gpu(c), *g, work)
    sadj.set_option("wave3d.zchunk", 0)
    torch.cuda.synchronize()
    return [to_host(t) for t in g]


# tile 64 x 32 (fp32: 128 x 32): edges of tiles, frames that leave the grid, axes without and with core tiles (fp64 from
# 68 x 132 cells on, fp32 from 68 x 260), the fewest planes that a wide plane needs to take three steps
SHAPES = {np.float64: [(897, 20, 24), (900, 31, 62), (897, 32, 64), (379, 33, 128), (281, 37, 150), (171, 35, 262), (137, 70, 136), (97, 65, 256),
                       (81, 68, 260), (71, 96, 196), (15, 33, 2048), (4, 500, 1024), (4, 1000, 1026)],
          np.float32: [(897, 33, 128), (449, 37, 152), (197, 68, 260), (197, 69, 264), (295, 35, 264), (90, 100, 660), (8, 1000, 1024)]}
CASES = [(d, s) for d in SHAPES for s in SHAPES[d]]


def _largest_sum(c, lams, nsteps):
    """The sum of the magnitudes of all terms that any value of the sweep is made of, at most."""
    inside = np.zeros(c.shape)
    inside[1:-1, 1:-1, 1:-1] = 1
    a, b, p, largest = np.abs(lams[0]) * inside, np.abs(lams[1]), np.abs(lams[2]), 0.0
    for _ in range(nsteps):
        q = c * a
        s = b + 2 * a + 6 * q
        for axis in range(3):                             # q is zero outside I: nothing comes round the ends
            s += np.roll(q, 1, axis) + np.roll(q, -1, axis)
        a, b, p = s * inside, p + a, 0.0
        largest = max(largest, s.max(), b.max())
    return largest


@pytest.mark.parametrize("dtype,shape", CASES)
def test_three_step_passes_are_exact_on_dyadic_data(sadj, shape, dtype):
    """fp64: c a multiple of 1/4, adjoints whole numbers up to 4: a step adds two bits below the point and at most four
    above, from three, so every sum of seven or eight steps is exact.  fp32: whole numbers, c 0 or 1, so few of them
    that no sum reaches 2^24.  So the GPU returns the oracle's numbers bit for bit."""
    if dtype == np.float64:
        c = np.clip(np.round(inputs.uniform(3, "c", shape, 0, 1) * 4) / 4, 0.0, 1.0)
        lams = [np.clip(np.round(4 * inputs.uniform(5, k, shape, -1, 1)), -4, 4) for k in ("r_bar", "u_bar", "u_prev_bar")]
    else:
        c = (inputs.uniform(3, "c", shape, 0, 1) < 0.04).astype(np.float64)
        lams = [np.round(0.8 * inputs.uniform(5, k, shape, -1, 1)) for k in ("r_bar", "u_bar", "u_prev_bar")]
        assert _largest_sum(c, lams, 7) < 2 ** 24
    inside = np.zeros(shape, dtype=bool)
    inside[1:-1, 1:-1, 1:-1] = True
    cn, l0 = np.where(inside, c, np.nan), np.where(inside, lams[0], np.nan)         # outside I: never used
    for nsteps in (7, 8) if dtype == np.float64 else (7,):
        want = oracle.wave_adjoint_steps(c, *lams, 1, nsteps)
        for zchunk in (0, 1, 3, 5, 7, 100) if nsteps == 7 else (0, 7):
            got = _run(sadj, nsteps, zchunk, cn.astype(dtype), [x.astype(dtype) for x in (l0, lams[1], lams[2])])
            for k in (nsteps % 3, (nsteps + 1) % 3):
                assert np.array_equal(got[k], want[k]), "buffer %d after %d steps, chunks of %d: %d cells differ" % (
                    k, nsteps, zchunk, int(np.sum(got[k] != want[k])))


@pytest.mark.parametrize("dtype,shape", [(np.float64, (897, 20, 24)), (np.float64, (171, 35, 264)), (np.float64, (81, 68, 260)),
                                         (np.float32, (449, 37, 152)), (np.float32, (197, 68, 260))])
def test_three_step_passes_match_the_oracle(sadj, shape, dtype):
    """Real-valued inputs within the rounding of the terms: each step adds at most 9 of them, so the relative
    error of a sweep stays below nsteps times the single-step tolerance of the largest value."""
    c = inputs.uniform(1, "c", shape, 0.01, 0.1).astype(dtype)
    lams = [inputs.uniform(2, k, shape, -1, 1).astype(dtype) for k in ("r_bar", "u_bar", "u_prev_bar")]
    for nsteps in (7, 11, 14):
        want = oracle.wave_adjoint_steps(c, *lams, 1, nsteps)
        for zchunk in (0, 9, 100):
            got = _run(sadj, nsteps, zchunk, c, lams)
            for k in (nsteps % 3, (nsteps + 1) % 3):
                g = got[k].astype(np.float64)
                assert np.isfinite(g).all()
                assert np.max(np.abs(g - want[k])) <= TOL[np.dtype(dtype)] * nsteps * max(np.max(np.abs(want[k])), 1e-300)


@pytest.mark.parametrize("dtype,shape", [(np.float64, (207, 35, 136)), (np.float64, (136, 35, 208)), (np.float64, (81, 68, 260)),
                                         (np.float64, (96, 100, 128)), (np.float32, (96, 130, 164)), (np.float32, (197, 68, 260))])
def test_options_that_move_work_change_no_bit(sadj, shape, dtype):
    """wave3d.zchunk, split, xcdmap, band and ldspad only move work between workgroups."""
    import torch
    c = to_gpu(inputs.uniform(1, "c", shape, 0.01, 0.1).astype(dtype))
    lams = [to_gpu(inputs.uniform(2, k, shape, -1, 1).astype(dtype)) for k in ("r_bar", "u_bar", "u_prev_bar")]
    nsteps, want = 9, None
    for name, value in [("wave3d.split", 0), ("wave3d.split", 1), ("wave3d.ldspad", -1), ("wave3d.ldspad", 4096), ("wave3d.xcdmap", 3),
                        ("wave3d.band", 1), ("wave3d.zchunk", 2), ("wave3d.zchunk", 5), ("wave3d.zchunk", 9), ("wave3d.zchunk", 100)]:
        g = [x.clone() for x in lams]
        sadj.set_option(name, value)
        sadj.sadj_adjoint_wave3d_steps_fused(1, nsteps, c, *g, torch.empty_like(c))
        sadj.set_option(name, 0)
        got = [g[nsteps % 3], g[(nsteps + 1) % 3]]
        want = want or got
        assert all(torch.equal(a, b) for a, b in zip(got, want)), (name, value)
