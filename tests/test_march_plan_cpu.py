"""Host-only test of the z cut of small grids: a grid whose tiles do not fill the chip is cut into chunks
shorter than 4R planes, as many as there are compute units for and no more."""
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
    assert info["workgroups"] <= CUS
    longest = max(ze - zs for _, _, zs, ze in tiles)
    # the longest chunk is as short as the compute units allow
    assert longest <= max(-(-nz // max(1, CUS // n_tiles)), 1)
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
