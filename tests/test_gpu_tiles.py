"""Tiles fitted to the cube (FP32 duals): widths that leave threads of a tile
idle (10 x 101, 31 x 33, 60 x 17, 45 x 3 and 135 x 1 pixels of 1024 threads),
widths in several slabs, tiles of one band and of all of them, rows and bands
left over, each with the chunk left to the library and with 8 bands asked for;
the same bits alone and in a batch.

The iterates follow the FP64 oracle. FP32 iterates round each of about 30
operations per iteration at 6e-8: 25 iterations stay below 1e-5."""
import numpy as np
import pytest

from gpu_helpers import announce, dev, f32, rel_l2, torch_cuda
from synth.cubes import SMALL_64x64x16, like, make_cube
from test_gpu_step import STATE, get_state

pytestmark = pytest.mark.gpu

# (N3, N1, N2)
SHAPES = [(5, 23, 101), (3, 29, 139), (2, 70, 17), (4, 200, 3), (2, 33, 33), (3, 140, 1), (1, 300, 2), (2, 2, 300),
          (16, 64, 64), (9, 50, 112), (33, 9, 112), (1, 1, 1), (70, 16, 48)]


def setup(shape, chunk, seed=41):
    import paper_2510_00562_amd as geo
    n3, n1, n2 = shape
    c = make_cube(like(SMALL_64x64x16, n1=n1, n2=n2, n3=n3, seed=seed, cells=5))
    v = f32(c["v"])
    dims, vd = geo.dims_of(shape), dev(v)
    p = geo.params(c["eps"], c["alpha"], c["beta"], omega=0.03, band_chunk=chunk)
    ws = geo.Workspace(geo.geo_workspace_size(dims, p))
    geo.geo_state_init(dims, p, vd, ws)
    return c, v, dims, vd, p, ws


@pytest.mark.parametrize("chunk", [0, 8])
@pytest.mark.parametrize("shape", SHAPES)
def test_fitted_tiles_follow_the_oracle(ora, shape, chunk):
    announce(f"fitted tiles {shape}, chunk {chunk}")
    torch_cuda()
    import paper_2510_00562_amd as geo
    c, v, dims, vd, p, ws = setup(shape, chunk)
    geo.geo_step(dims, p, vd, ws, 25)
    got = get_state(geo, dims, p, ws, vd, shape)
    S = ora.Solver(v, c["eps"], c["alpha"], c["beta"], omega=0.03)
    S.step(25)
    for name in ("u", "s", "t"):
        want = S.state[name]
        if np.linalg.norm(want) > 0:
            assert rel_l2(got[name], want) <= 1e-5, name
        else:
            assert not got[name].any(), name


@pytest.mark.parametrize("chunk", [0, 16])
def test_fitted_tiles_in_a_batch(chunk):
    announce(f"fitted tiles in a batch, chunk {chunk}")
    torch_cuda()
    import paper_2510_00562_amd as geo
    st = [setup(s, chunk) for s in SHAPES[:10]]
    table = geo.Workspace(geo.geo_batch_table_size(len(st)))
    geo.geo_batch_step([x[2] for x in st], [x[4] for x in st], [x[3] for x in st], [x[5] for x in st], table, 20,
                       use_graph=True)
    for shape, (_, _, dims, vd, p, ws) in zip(SHAPES, st):
        batch = get_state(geo, dims, p, ws, vd, shape)
        geo.geo_state_init(dims, p, vd, ws)
        geo.geo_step(dims, p, vd, ws, 20)
        solo = get_state(geo, dims, p, ws, vd, shape)
        for name in STATE:
            assert np.array_equal(solo[name], batch[name]), (shape, name)
