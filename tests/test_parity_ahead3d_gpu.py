"""GPU test of the 3-D march whose requests run ahead (grids that do not fill the chip): the wave adjoint in every form against
the one-cell tiles of the other kernel, bit for bit, at the edges of tiles, vectors and chunks; against the oracle; NaN outside
I; arrays aligned to their elements only; a grid large enough for the streaming accesses."""
import numpy as np
import pytest

import inputs
import oracle
from parity import to_gpu, to_host

pytestmark = pytest.mark.gpu

# below, at and beyond tiles of 32 x 16, 64 x 16, 128 x 16 and 64 x 32 cells; rows of every length modulo 4; one plane per chunk and several
SHAPES = [(0, 0, 0), (13, 16, 32), (10, 17, 33), (31, 15, 66), (20, 33, 127), (9, 16, 129), (40, 31, 64), (150, 49, 95), (12, 300, 258)]


@pytest.fixture
def sadj():
    import paper_1907_02818_amd as lib
    lib.load()
    yield lib
    lib.set_option("wave3d.variant", 0)


def _shape(shape, radius):
    return tuple(max(n, 2 * radius + 1) for n in shape)


def _placed(torch, x, offset):
    """x in an array that starts `offset` elements behind an aligned address."""
    flat = torch.empty(x.numel() + offset, dtype=x.dtype, device="cuda")[offset:]
    return flat.view(x.shape).copy_(x)


def _calls(lib, torch, radius, c, a, b, p, offset):
    c, a = _placed(torch, c, offset), _placed(torch, a, offset)
    new = lambda x: _placed(torch, x, offset)   # noqa: E731
    out = [new(b), new(b), new(p), new(a), new(b), new(p), new(a), new(b), new(p)]
    lib.sadj_adjoint_wave3d(radius, c, a, out[0])
    lib.sadj_adjoint_wave3d(radius, c, a, out[1], out[2])
    lib.sadj_adjoint_wave3d_steps(radius, 2, c, *out[3:6])       # u_prev_bar accumulated, then assigned by the last step
    lib.sadj_adjoint_wave3d_steps(radius, 4, c, *out[6:9])       # with middle steps
    return out


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("radius", [1, 2, 3, 4])
def test_same_bits_as_the_one_cell_tiles(sadj, radius, dtype):
    import torch
    for k, shape in enumerate(SHAPES):
        shape = _shape(shape, radius)
        c, a, b, p = (to_gpu(inputs.uniform(k, n, shape, -1, 1).astype(dtype)) for n in ("c", "r_bar", "u_bar", "u_prev_bar"))
        got = _calls(sadj, torch, radius, c, a, b, p, k % 2)
        sadj.set_option("wave3d.variant", 3)
        want = _calls(sadj, torch, radius, c, a, b, p, k % 2)
        sadj.set_option("wave3d.variant", 0)
        for i, (x, y) in enumerate(zip(got, want)):
            assert torch.equal(x, y), (shape, i)


@pytest.mark.parametrize("shape,dtype", [((203, 245, 250), np.float64), ((300, 290, 290), np.float32), ((301, 290, 292), np.float32)])
def test_same_bits_with_streaming_accesses(sadj, shape, dtype):
    import torch
    g = torch.Generator(device="cuda").manual_seed(3)
    tt = torch.float64 if dtype == np.float64 else torch.float32
    c, a, b, p = (torch.empty(shape, device="cuda", dtype=tt).uniform_(-1, 1, generator=g) for _ in range(4))
    got = _calls(sadj, torch, 2, c, a, b, p, 0)
    sadj.set_option("wave3d.variant", 3)
    want = _calls(sadj, torch, 2, c, a, b, p, 0)
    for i, (x, y) in enumerate(zip(got, want)):
        assert torch.equal(x, y), i


@pytest.mark.parametrize("radius,shape", [(1, (11, 18, 35)), (2, (9, 20, 67)), (3, (16, 21, 130)), (4, (19, 17, 34))])
def test_against_the_oracle_with_nan_outside_the_iteration_space(sadj, radius, shape):
    d = inputs.config_inputs("wave3d_r4", shape=shape, seed=radius, c_mode="iid")
    inside = np.zeros(shape, bool)
    inside[tuple(slice(radius, n - radius) for n in shape)] = True
    want, want_p, scale = oracle.wave_adjoint(d["c"], d["r_bar"], d["u_bar"], radius, u_prev_bar=d["u_prev_bar"], want_scale=True)
    c, a = (np.where(inside, d[k], np.nan) for k in ("c", "r_bar"))
    ub, pb = to_gpu(d["u_bar"]), to_gpu(d["u_prev_bar"])
    sadj.sadj_adjoint_wave3d(radius, to_gpu(c), to_gpu(a), ub, pb)
    # a cell is a sum of at most 6R + 3 products: as many roundings of the sum of their magnitudes, and those of the oracle's
    bound = 2 * (6 * radius + 4) * np.finfo(np.float64).eps * (scale + np.abs(d["u_bar"]))
    assert np.all(np.abs(to_host(ub) - want) <= bound)
    assert np.array_equal(to_host(pb), want_p)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("radius", [1, 2, 3, 4])
def test_star_is_exact_on_dyadic_data(sadj, radius, dtype):
    """Weights and c multiples of 1/4 below 2, fields whole numbers up to 4: every product is a multiple of 1/16 and the at most
    25 terms stay below 512, 13 bits in all, so fp32 is exact as well.  NaN where values must not be read."""
    import torch
    for k, shape in enumerate(SHAPES):
        shape = _shape(shape, radius)
        w = np.round(inputs.uniform(2, "aux", (1 + 6 * radius,), -2, 2) * 4) / 4
        c = np.round(inputs.uniform(3, "c", shape, 0, 1) * 4) / 4
        u, rb, ub = (np.round(4 * inputs.uniform(5, n, shape, -1, 1)) for n in ("u", "r_bar", "u_bar"))
        m = np.zeros(shape, bool)
        m[tuple(slice(radius, n - radius) for n in shape)] = True
        put = lambda x: _placed(torch, to_gpu(x.astype(dtype)), k % 2)   # noqa: E731
        got = put(ub)
        sadj.sadj_adjoint_star3d(radius, w, put(np.where(m, c, np.nan)), put(np.where(m, rb, np.nan)), got)
        assert np.array_equal(to_host(got).astype(np.float64), oracle.star3d_adjoint(w, c, rb, ub, radius)[0]), shape
        r = put(np.full(shape, 7.0))
        sadj.sadj_primal_star3d(radius, w, put(u), put(np.where(m, c, np.nan)), r)
        assert np.array_equal(to_host(r).astype(np.float64)[m], oracle.star3d_primal(w, u, c, radius)[m]), shape
        assert (to_host(r)[~m] == 7).all(), shape


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("radius", [1, 2, 3, 4])
def test_wave_primal_against_the_oracle(sadj, radius, dtype):
    import torch
    from parity import wave_primal_scale
    for k, shape in enumerate(SHAPES):
        shape = _shape(shape, radius)
        d = inputs.wave_inputs(shape, 0.01, 0.1, seed=k, dtype=dtype, c_mode="iid")
        m = np.zeros(shape, bool)
        m[tuple(slice(radius, n - radius) for n in shape)] = True
        put = lambda x: _placed(torch, to_gpu(x.astype(dtype)), k % 2)   # noqa: E731
        r = put(np.full(shape, 7.0))
        sadj.sadj_primal_wave3d(radius, put(d["u"]), put(np.where(m, d["u_prev"], np.nan)), put(np.where(m, d["c"], np.nan)), r)
        want = oracle.wave_primal(d["u"], d["u_prev"], d["c"], radius)
        scale = wave_primal_scale(d["u"], d["u_prev"], d["c"], radius)
        # as many roundings as terms, of the sum of their magnitudes
        bound = (6 * radius + 6) * np.finfo(dtype).eps * scale
        got = to_host(r).astype(np.float64)
        assert np.all(np.abs(got - want)[m] <= bound[m]), shape
        assert (got[~m] == 7).all(), shape
