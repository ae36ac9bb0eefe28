"""GPU tests of the kernels that larger 3-D grids run, on small arrays: option "wave3d.ahead" 1 sends every grid to them, and the
lists of shapes of the parity tests, whose grids otherwise take the march with its requests ahead, go through them as well."""
import numpy as np
import pytest

import inputs
import test_parity_ahead3d_gpu as ahead
import test_parity_star3d_gpu as star
import test_parity_wave3d_gpu as wave
import test_parity_wave_middle_steps_gpu as middle
from parity import to_gpu

pytestmark = pytest.mark.gpu

DTYPES = [np.float64, np.float32]


def _rows(test):
    """The argument lists of a test's parametrize mark whose names are not `dtype`."""
    return [m for m in test.pytestmark if m.name == "parametrize" and m.args[0] != "dtype"][0].args[1]


@pytest.fixture
def sadj():
    import paper_1907_02818_amd as lib
    lib.load()
    lib.set_option("wave3d.ahead", 1)
    yield lib
    for name in ("ahead", "zchunk", "split", "xcdmap", "band", "ldspad"):
        lib.set_option("wave3d." + name, 0)


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("radius,shape", wave.SMALL)
def test_wave_adjoint_and_primal(sadj, radius, shape, dtype):
    wave.test_adjoint_small(sadj, radius, shape, dtype)
    wave.test_primal_small(sadj, radius, shape, dtype)


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("radius,shape", _rows(wave.test_unaligned_rows_take_wide_tiles))
def test_wave_rows_that_are_not_line_multiples(sadj, radius, shape, dtype):
    wave.test_unaligned_rows_take_wide_tiles(sadj, radius, shape, dtype)


@pytest.mark.parametrize("case", range(24))
def test_wave_on_drawn_shapes_and_options(sadj, case):
    wave.test_adjoint_and_primal_on_drawn_shapes_and_options(sadj, case)


@pytest.mark.parametrize("dtype", DTYPES)
def test_wave_odd_extent_and_unaligned_arrays(sadj, dtype):
    wave.test_odd_extent_and_unaligned_arrays_take_the_scalar_shape(sadj, dtype)


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("radius,shape", _rows(wave.test_cutting_and_placing_the_work_differently_changes_no_bit))
def test_wave_cutting_the_work_differently_changes_no_bit(sadj, radius, shape, dtype):
    wave.test_cutting_and_placing_the_work_differently_changes_no_bit(sadj, radius, shape, dtype)


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("radius,shape", _rows(middle.test_middle_steps_equal_single_calls_bitwise))
def test_wave_middle_steps(sadj, radius, shape, dtype):
    middle.test_middle_steps_equal_single_calls_bitwise(sadj, radius, shape, dtype)


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("radius,shape", _rows(middle.test_middle_steps_of_long_marches))
def test_wave_middle_steps_of_long_marches(sadj, radius, shape, dtype):
    middle.test_middle_steps_of_long_marches(sadj, radius, shape, dtype)


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("radius,shape", star.CASES)
def test_star_adjoint_and_primal(sadj, radius, shape, dtype):
    star.test_star_adjoint_and_primal(sadj, 0, radius, shape, dtype)


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("radius", [1, 2, 3, 4])
def test_star_is_exact_on_dyadic_data_and_primal_keeps_its_bounds(sadj, radius, dtype):
    """At the edges of tiles, on arrays aligned to their elements only, NaN where values must not be read."""
    ahead.test_star_is_exact_on_dyadic_data(sadj, radius, dtype)
    ahead.test_wave_primal_against_the_oracle(sadj, radius, dtype)


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("radius", [1, 2, 3, 4])
def test_wave_adjoint_has_the_bits_of_the_march_ahead(sadj, radius, dtype):
    """All forms (u_bar alone, u_prev_bar accumulated or assigned, middle steps), aligned and unaligned arrays."""
    import torch
    for k, shape in enumerate(ahead.SHAPES):
        shape = ahead._shape(shape, radius)
        c, a, b, p = (to_gpu(inputs.uniform(k, n, shape, -1, 1).astype(dtype)) for n in ("c", "r_bar", "u_bar", "u_prev_bar"))
        sadj.set_option("wave3d.ahead", 1)
        got = ahead._calls(sadj, torch, radius, c, a, b, p, k % 2)
        sadj.set_option("wave3d.ahead", 0)
        want = ahead._calls(sadj, torch, radius, c, a, b, p, k % 2)
        for i, (x, y) in enumerate(zip(got, want)):
            assert torch.equal(x, y), (shape, i)
