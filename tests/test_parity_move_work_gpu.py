"""GPU test of the options that only move work between workgroups (wave3d.zchunk, split, xcdmap, band, ldspad): every bit of
the single 3-D calls stays as it is, in short and in long marches, in tiles of every shape that small grids take."""
import numpy as np
import pytest

import inputs
from parity import to_gpu

pytestmark = pytest.mark.gpu

OPTIONS = [("zchunk", 1), ("zchunk", 3), ("zchunk", 17), ("zchunk", 1000), ("split", 1), ("ldspad", -1), ("ldspad", 2048), ("xcdmap", 3), ("band", 2)]


@pytest.fixture
def sadj():
    import paper_1907_02818_amd as lib
    lib.load()
    yield lib
    lib.set_option("wave3d.order", 0)
    for name, _ in OPTIONS:
        lib.set_option("wave3d." + name, 0)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("radius,shape", [(1, (24, 40, 72)), (1, (60, 33, 131)), (2, (40, 35, 132)), (3, (31, 20, 64)), (4, (9, 9, 9)), (4, (40, 40, 40)),
                                          (4, (98, 34, 52)), (4, (45, 70, 260)), (4, (63, 81, 97))])
def test_no_bit_changes(sadj, radius, shape, dtype):
    import torch
    c, a, b, p = (to_gpu(inputs.uniform(5, k, shape, -1, 1).astype(dtype)) for k in ("c", "r_bar", "u_bar", "u_prev_bar"))
    w = list(inputs.uniform(2, "aux", (1 + 6 * radius,), -1, 1))
    wb = inputs.uniform(2, "u", (3, 3, 3), -1, 1)

    def calls():
        out = [b.clone() for _ in range(6 if radius > 1 else 8)] + [p.clone()]
        sadj.sadj_adjoint_wave3d(radius, c, a, out[0])
        sadj.sadj_adjoint_wave3d(radius, c, a, out[1], out[-1])
        sadj.sadj_primal_wave3d(radius, a, p, c, out[2])
        sadj.sadj_adjoint_star3d(radius, w, c, a, out[3])
        sadj.sadj_primal_star3d(radius, w, a, c, out[4])
        sadj.set_option("wave3d.order", 1)
        sadj.sadj_adjoint_wave3d(radius, c, a, out[5])
        sadj.set_option("wave3d.order", 0)
        if radius == 1:
            sadj.sadj_adjoint_box(wb, c, a, out[6])
            sadj.sadj_primal_box(wb, a, c, out[7])
        return out

    want = calls()
    for name, value in OPTIONS:
        sadj.set_option("wave3d." + name, value)
        got = calls()
        sadj.set_option("wave3d." + name, 0)
        for i, (x, y) in enumerate(zip(got, want)):
            assert torch.equal(x, y), (name, value, i)
