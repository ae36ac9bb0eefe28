"""Host-only test of the z cut of small grids: a grid whose tiles do not fill the chip is cut into chunks
shorter than 4R planes, as many as there are workgroups resident and no more, and takes 32 x 16 tiles,
two per compute unit, where those march for a shorter time."""
import pytest

# without a GPU the planner assumes this many compute units
CUS = 256


def _plan(dtype_code, radius, shape):
    import paper_1907_02818_amd as lib
    nz, ny, nx = shape
    return lib.sadj_describe_wave3d_plan(dtype_code, radius, nx, ny, nz)


@pytest.mark.parametrize("dtype_code", [0, 1])
@pytest.mark.parametrize("radius", [1, 2, 4])
@pytest.mark.parametrize("shape", [(9, 9, 9), (40, 40, 40), (80, 96, 112), (101, 99, 97), (128, 128, 128), (300, 20, 64), (17, 400, 512)])
def test_small_grids_fill_the_chip_in_one_round(dtype_code, radius, shape):
    torch = pytest.importorskip("torch")
    if torch.cuda.is_available():
        pytest.skip("plans depend on the device's compute units; this test counts on the default")
    info, tiles = _plan(dtype_code, radius, shape)
    nz = shape[0]
    n_tiles = info["ntx"] * info["nty"]
    resident = 2 * CUS if (info["tile_w"], info["tile_h"]) == (32, 16) else CUS
    assert info["workgroups"] <= resident
    longest = max(ze - zs for _, _, zs, ze in tiles)
    # the longest chunk is as short as the resident workgroups allow
    assert longest <= max(-(-nz // max(1, resident // n_tiles)), 1)
    seen = {}
    for tx, ty, zs, ze in tiles:
        seen.setdefault((tx, ty), []).append((zs, ze))
    assert len(seen) == n_tiles
    for spans in seen.values():
        spans.sort()
        assert spans[0][0] == 0 and spans[-1][1] == nz
        assert all(a[1] == b[0] and a[0] < a[1] for a, b in zip(spans, spans[1:]))


def test_larger_grids_keep_chunks_of_at_least_four_radii():
    info, tiles = _plan(1, 4, (256, 256, 256))
    assert min(ze - zs for _, _, zs, ze in tiles) >= 16 or info["workgroups"] <= CUS
    info, tiles = _plan(1, 4, (200, 1000, 1000))
    assert min(ze - zs for _, _, zs, ze in tiles) >= 16


@pytest.mark.parametrize("dtype_code,radius,shape,small", [(1, 4, (40, 40, 40), True), (1, 4, (80, 96, 112), True), (1, 1, (80, 96, 112), False),
                                                           (0, 4, (128, 128, 128), True), (1, 4, (160, 180, 200), False),
                                                           (1, 4, (256, 256, 256), False), (1, 4, (20, 37, 250), False)])
def test_which_grids_take_small_tiles(dtype_code, radius, shape, small):
    torch = pytest.importorskip("torch")
    if torch.cuda.is_available():
        pytest.skip("plans depend on the device's compute units; this test counts on the default")
    info, _ = _plan(dtype_code, radius, shape)
    assert ((info["tile_w"], info["tile_h"]) == (32, 16)) == small


@pytest.mark.parametrize("radius,shape,small", [(1, (73, 174, 61), False), (1, (44, 28, 71), False), (2, (117, 161, 49), False),
                                                (3, (46, 39, 83), True), (4, (37, 178, 39), True), (4, (37, 178, 40), True)])
def test_small_tiles_are_priced_against_the_shape_that_would_run(radius, shape, small):
    """fp32 rows that are not whole vectors otherwise run in 64 x 32 tiles, which small tiles beat only at larger radii."""
    torch = pytest.importorskip("torch")
    if torch.cuda.is_available():
        pytest.skip("plans depend on the device's compute units; this test counts on the default")
    info, _ = _plan(0, radius, shape)
    assert (info["tile_w"], info["tile_h"]) == ((32, 16) if small else (64, 32))
