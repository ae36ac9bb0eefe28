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
