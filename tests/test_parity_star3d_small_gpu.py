"""GPU parity of the radius-4 star in 32 x 16 tiles, which small grids take: exact on dyadic data at the
edges of those tiles, NaN where values must not be read."""
import numpy as np
import pytest

import inputs
import oracle
from jacobians import interior_mask
from parity import to_gpu, to_host

pytestmark = pytest.mark.gpu


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
