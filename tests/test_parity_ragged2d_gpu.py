"""GPU parity of the 2-D tile kernels where rows or arrays are not aligned to whole 16-byte vectors: every
remainder of nx modulo the vector length at the edges of a tile, the smallest grids, arrays that start
one element off, and sentinels around the arrays that a kernel must not touch."""
import numpy as np
import pytest

import inputs
import oracle
from parity import assert_close, to_host, wave_primal_scale

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sadj():
    import paper_1907_02818_amd as lib
    lib.load()
    return lib


class _Arrays:
    """Device arrays that start `shift` elements into an allocation filled with a sentinel."""

    def __init__(self, shift):
        self.shift, self.all = shift, []

    def put(self, a):
        import torch
        buf = torch.full((a.size + 16 + self.shift,), 7.5, dtype=torch.from_numpy(a[:1]).dtype, device="cuda")
        t = buf[8 + self.shift:8 + self.shift + a.size].view(a.shape)
        t.copy_(torch.from_numpy(np.ascontiguousarray(a)))
        self.all.append((buf, a.size))
        return t

    def check(self):
        for buf, n in self.all:
            b = to_host(buf)
            lo = 8 + self.shift
            assert (b[:lo] == 7.5).all() and (b[lo + n:] == 7.5).all()


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("nx", [3, 4, 5, 6, 7, 63, 65, 66, 67, 127, 128, 129, 130, 131, 191, 193, 257, 258, 259])
@pytest.mark.parametrize("ny,shift", [(3, 0), (9, 1), (20, 0), (33, 3)])
def test_ragged_rows(sadj, nx, ny, shift, dtype):
    import torch
    shape = (ny, nx)
    d = {k: inputs.uniform(nx + ny, k, shape, -1, 1).astype(dtype) for k in ("u", "u_prev", "r_bar", "u_bar", "u_prev_bar")}
    c = inputs.uniform(1, "c", shape, 0.01, 0.2).astype(dtype)
    m = np.zeros(shape, dtype=bool)
    m[1:-1, 1:-1] = True
    cn, rn = np.where(m, c, np.nan).astype(dtype), np.where(m, d["r_bar"], np.nan).astype(dtype)   # outside I: never used
    for both in (False, True):
        A = _Arrays(shift)
        ub, pb = A.put(d["u_bar"]), A.put(d["u_prev_bar"])
        sadj.sadj_adjoint_wave2d(A.put(cn), A.put(rn), ub, pb if both else None)
        torch.cuda.synchronize()
        A.check()
        wu, wp, scale = oracle.wave_adjoint(c, d["r_bar"], d["u_bar"], 1, u_prev_bar=d["u_prev_bar"], want_scale=True)
        assert_close(to_host(ub), wu, scale + np.abs(d["u_bar"].astype(np.float64)), dtype, "u_bar")
        want_p = wp if both else d["u_prev_bar"]
        assert_close(to_host(pb), want_p, np.abs(d["u_prev_bar"].astype(np.float64)) + 1.0, dtype, "u_prev_bar")
    A = _Arrays(shift)
    r = A.put(d["r_bar"])
    sadj.sadj_primal_wave2d(A.put(d["u"]), A.put(d["u_prev"]), A.put(cn), r)
    torch.cuda.synchronize()
    A.check()
    want = oracle.wave_primal(d["u"], d["u_prev"], c, 1, r_init=d["r_bar"])
    got = to_host(r)
    assert np.array_equal(got[~m], d["r_bar"][~m])
    assert_close(got[m], want[m], wave_primal_scale(d["u"], d["u_prev"], c, 1)[m], dtype, "r")
    w = np.linspace(-1, 1, 9).reshape(3, 3)
    wt = w.astype(dtype).astype(np.float64)
    A = _Arrays(shift)
    ub, r = A.put(d["u_bar"]), A.put(d["r_bar"])
    sadj.sadj_adjoint_box(w, A.put(cn), A.put(rn), ub)
    sadj.sadj_primal_box(w, A.put(d["u"]), A.put(cn), r)
    torch.cuda.synchronize()
    A.check()
    wu, scale = oracle.box_adjoint(wt, c, d["r_bar"], d["u_bar"], want_scale=True)[:2]
    assert_close(to_host(ub), wu, scale + np.abs(d["u_bar"].astype(np.float64)), dtype, "box u_bar")
    got = to_host(r)
    want = oracle.box_primal(wt, d["u"], c, r_init=d["r_bar"])
    assert np.array_equal(got[~m], d["r_bar"][~m])
    # nine products and a factor of at most 0.2: the sum of their magnitudes is below 9 * 0.2
    assert_close(got[m], want[m], np.full(int(m.sum()), 1.8), dtype, "box r")


def test_large_ragged_arrays_with_u_prev_bar(sadj):
    """The four arrays exceed 256 MB, where u_bar and u_prev_bar take regular accesses: a float64 reference
    of whole-array torch operations."""
    import torch
    ny, nx = 2100, 4099
    g = torch.Generator(device="cuda").manual_seed(1)
    rnd = lambda: torch.rand((ny, nx), generator=g, dtype=torch.float64, device="cuda") - 0.5   # noqa: E731
    c, r, u, p = rnd(), rnd(), rnd(), rnd()
    q = torch.zeros_like(c)
    q[1:-1, 1:-1] = c[1:-1, 1:-1] * r[1:-1, 1:-1]
    wu = u - 4 * q
    wu[:, 1:] += q[:, :-1]
    wu[:, :-1] += q[:, 1:]
    wu[1:] += q[:-1]
    wu[:-1] += q[1:]
    wu[1:-1, 1:-1] += 2 * r[1:-1, 1:-1]
    wp = p.clone()
    wp[1:-1, 1:-1] -= r[1:-1, 1:-1]
    sadj.sadj_adjoint_wave2d(c, r, u, p)
    # seven terms of magnitude below 2: rounding below 7 * 2 * 2^-53 each
    assert (u - wu).abs().max().item() <= 7 * 2 * 2.0 ** -52
    assert torch.equal(p, wp)


def test_large_ragged_fp32_arrays_with_u_prev_bar(sadj):
    """The same in fp32, where the four arrays exceed 256 MB from 4097 x 4097 cells on; reference in float64."""
    import torch
    ny, nx = 4097, 4099
    g = torch.Generator(device="cuda").manual_seed(1)
    rnd = lambda: torch.rand((ny, nx), generator=g, dtype=torch.float32, device="cuda") - 0.5   # noqa: E731
    c, r, u, p = rnd(), rnd(), rnd(), rnd()
    q = torch.zeros((ny, nx), dtype=torch.float64, device="cuda")
    q[1:-1, 1:-1] = c[1:-1, 1:-1].double() * r[1:-1, 1:-1].double()
    wu = u.double() - 4 * q
    wu[:, 1:] += q[:, :-1]
    wu[:, :-1] += q[:, 1:]
    wu[1:] += q[:-1]
    wu[:-1] += q[1:]
    wu[1:-1, 1:-1] += 2 * r[1:-1, 1:-1].double()
    wp = p.double()
    wp[1:-1, 1:-1] -= r[1:-1, 1:-1].double()
    sadj.sadj_adjoint_wave2d(c, r, u, p)
    # as above, with the products rounded to fp32 first: eight terms of magnitude below 2, rounding below 2 * 2^-24 each; one
    # subtraction of numbers below 1 in u_prev_bar
    assert (u.double() - wu).abs().max().item() <= 8 * 2 * 2.0 ** -23
    assert (p.double() - wp).abs().max().item() <= 2.0 ** -24
