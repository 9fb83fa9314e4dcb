"""The query of the tiles that the sweep runs (host side, no GPU): for every cube,
storage and request they cover the cube, fit a workgroup and the workspace, keep the
bands asked for (unless 8 x 128 tiles of them are more than 4096), and with BF16 duals are as many as the nominal geometry says."""
import ctypes

import pytest

SHAPES = [(16, 64, 64), (64, 128, 128), (198, 120, 120), (360, 100, 100), (156, 131, 139), (128, 256, 256),
          (224, 512, 512), (4, 2048, 2048), (100000, 1, 1), (20000, 2, 3), (5000, 16, 16), (300, 4096, 1),
          (300, 1, 4096), (7, 13, 19), (1, 1, 1), (33, 17, 16)]


@pytest.mark.parametrize("dual", [0, 1])
@pytest.mark.parametrize("shape", SHAPES)
def test_tiles_cover_the_cube(shape, dual):
    import paper_2510_00562_amd as geo
    n3, n1, n2 = shape
    d = geo.dims_of(shape)
    for blocks in (1, 256, 304):
        for requested in (0, 5, 16, 64, 300000):
            kc, tiles, rows, cols = geo.geo_sweep_tiles(d, requested, blocks, dual)
            assert tiles == -(-n1 // rows) * -(-n2 // cols) * -(-n3 // kc)
            assert rows * cols <= 1024 and rows + cols <= 136 and cols <= 128
            assert tiles <= geo.geo_workspace_tiles(d, dual) and tiles <= 4096
            asked = max(requested, 8)
            if requested and -(-n1 // 8) * -(-n2 // 128) * -(-n3 // asked) <= 4096:
                assert kc == asked
            if dual:
                assert (kc, tiles) == geo.geo_sweep_geometry(d, requested, blocks, dual)[:2]


@pytest.mark.parametrize("shape,want", [
    # one band each of 16 x 64 pixels; all 224 bands of 8 x 128 pixels; the whole
    # width of 120 columns; one round of 4 x 256 workgroups over a spectrum
    ((16, 64, 64), (1, 64, 16, 64)),
    ((224, 512, 512), (224, 256, 8, 128)),
    ((100000, 1, 1), (98, 1021, 1, 1)),
    ((5000, 16, 16), (5, 1000, 16, 16)),
])
def test_tiles_of_known_cubes(shape, want):
    import paper_2510_00562_amd as geo
    assert geo.geo_sweep_tiles(geo.dims_of(shape), 0, 256) == want


def test_argument_checks():
    import paper_2510_00562_amd as geo
    L = geo.lib()
    x = ctypes.c_int32()
    out = [ctypes.byref(x)] * 4
    assert L.geo_sweep_tiles(geo.geo_dims(0, 4, 4), 0, 8, 256, *out) == -1
    assert L.geo_sweep_tiles(geo.geo_dims(4, 4, 4), 5, 8, 256, *out) == -1
    assert L.geo_sweep_tiles(geo.geo_dims(4, 4, 4), 0, -1, 256, *out) == -1
    assert L.geo_sweep_tiles(geo.geo_dims(4, 4, 4), 0, 8, 0, *out) == -1
    assert L.geo_sweep_tiles(geo.geo_dims(4, 4, 4), 0, 8, 256, None, *out[1:]) == -1
