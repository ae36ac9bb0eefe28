"""GPU parity of the radius-4 star on small grids, which take 32 x 16 tiles or wider ones of 16 rows (the march with its requests
ahead): exact on dyadic data at the edges of those tiles, NaN where values must not be read."""
import numpy as np
import pytest

import inputs
import oracle
from jacobians import interior_mask
from parity import to_gpu, to_host

pytestmark = pytest.mark.gpu


@pytest.fixture
def sadj_options():
    """Leaves the options as they are by default, whatever happens in between."""
    import paper_1907_02818_amd as lib
    yield
    for name in ("zchunk", "split", "xcdmap", "band", "ldspad"):
        lib.set_option("wave3d." + name, 0)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("shape", [(9, 9, 9), (24, 16, 32), (25, 17, 33), (40, 25, 41), (64, 33, 64), (70, 48, 97), (101, 34, 96)])
def test_small_tiles_are_exact_on_dyadic_data(shape, dtype):
    """Weights and c multiples of 1/4 below 2, fields whole numbers up to 4: every product is a multiple of 1/16
    and the 25 terms stay below 512, 13 bits in all, so fp32 is exact as well."""
    import paper_1907_02818_amd as sadj
    w = np.round(inputs.uniform(2, "aux", (25,), -2, 2) * 4) / 4
    c = np.round(inputs.uniform(3, "c", shape, 0, 1) * 4) / 4
    u, rb, ub = (np.round(4 * inputs.uniform(5, k, shape, -1, 1)) for k in ("u", "r_bar", "u_bar"))
    m = interior_mask(shape, 4)
    got = to_gpu(ub.astype(dtype))
    sadj.sadj_adjoint_star3d(4, w, to_gpu(np.where(m, c, np.nan).astype(dtype)), to_gpu(np.where(m, rb, np.nan).astype(dtype)), got)
    assert np.array_equal(to_host(got).astype(np.float64), oracle.star3d_adjoint(w, c, rb, ub, 4)[0])
    r = to_gpu(np.full(shape, 7, dtype=dtype))
    sadj.sadj_primal_star3d(4, w, to_gpu(u.astype(dtype)), to_gpu(np.where(m, c, np.nan).astype(dtype)), r)
    assert np.array_equal(to_host(r).astype(np.float64)[m], oracle.star3d_primal(w, u, c, 4)[m])
    assert (to_host(r)[~m] == 7).all()


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("shape", [(9, 21, 40), (16, 35, 80), (63, 81, 96), (98, 34, 52), (40, 40, 41)])
def test_options_that_move_work_change_no_bit(sadj_options, shape, dtype):
    """wave3d.zchunk, split, xcdmap, band and ldspad only move work between workgroups."""
    import torch
    import paper_1907_02818_amd as sadj
    w = list(inputs.uniform(2, "aux", (25,), -1, 1))
    c, x, ub = (to_gpu(inputs.uniform(5, k, shape, -1, 1).astype(dtype)) for k in ("c", "r_bar", "u_bar"))
    want = None
    for name, value in [("wave3d.split", 0), ("wave3d.split", 1), ("wave3d.ldspad", -1), ("wave3d.ldspad", 2048), ("wave3d.xcdmap", 3),
                        ("wave3d.band", 2), ("wave3d.zchunk", 1), ("wave3d.zchunk", 3), ("wave3d.zchunk", 50)]:
        got = [ub.clone(), ub.clone()]
        sadj.set_option(name, value)
        sadj.sadj_adjoint_star3d(4, w, c, x, got[0])
        sadj.sadj_primal_star3d(4, w, x, c, got[1])
        sadj.set_option(name, 0)
        want = want or got
        assert all(torch.equal(a, b) for a, b in zip(got, want)), (name, value)


def _fp32_error_of_an_in_plane_sum(w, u, c):
    """2-norm error, over that of the result, of the fp32 radius-1 primal whose in-plane terms are one sum that starts at the
    centre (products of two floats are exact in fp64, so its fused multiply-adds are fp64 operations rounded to fp32), and the exact result."""
    def rounded(x):
        return x.astype(np.float32).astype(np.float64)

    at = [u[1:-1, 1:-1, 1:-1]] + [u[tuple(slice(1 + (o if a == d else 0), n - 1 + (o if a == d else 0)) for a, n in enumerate(u.shape))]
                                  for d in (2, 1, 0) for o in (-1, 1)]
    t = rounded(w[0] * at[0])
    for k in (1, 2, 3, 4):
        t = rounded(w[k] * at[k] + t)
    t = rounded(w[6] * at[6] + rounded(rounded(w[5] * at[5]) + t))
    c = c[1:-1, 1:-1, 1:-1]
    exact = c * sum(a * b for a, b in zip(w, at))
    return np.linalg.norm(rounded(c * t) - exact) / np.linalg.norm(exact), exact


@pytest.mark.parametrize("kind", ["random", "one-sided", "laplacian"])
def test_radius_1_rounds_no_worse_than_an_in_plane_sum(kind):
    """24 sets of weights, geometric mean: the sum of seven roundings stays below the eight of the other order (0.99, 0.97 and 0.66
    of it by emulation; nine, with each axis summed by itself, 1.01, 1.06 and 0.80)."""
    import paper_1907_02818_amd as sadj
    shape, ratio = (26, 40, 64), []
    for seed in range(24):
        rng = np.random.default_rng(seed)
        w = rng.uniform(-0.5, 0.5, 7) if kind != "laplacian" else np.array([-6.0, 1, 1, 1, 1, 1, 1])
        if kind == "one-sided":
            w[2::2] = 0
        w = w.astype(np.float32).astype(np.float64)
        u, c = rng.uniform(-1, 1, shape).astype(np.float32), rng.uniform(0.03, 0.23, shape).astype(np.float32)
        r = to_gpu(np.zeros(shape, dtype=np.float32))
        sadj.sadj_primal_star3d(1, list(w), to_gpu(u), to_gpu(c), r)
        other, exact = _fp32_error_of_an_in_plane_sum(w, u.astype(np.float64), c.astype(np.float64))
        ratio.append(np.linalg.norm(to_host(r)[1:-1, 1:-1, 1:-1].astype(np.float64) - exact) / np.linalg.norm(exact) / other)
    assert np.exp(np.log(ratio).mean()) <= 1.0
