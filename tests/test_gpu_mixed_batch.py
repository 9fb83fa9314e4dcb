"""How the tiles of a batch are dealt to the XCDs and their blocks: fewer tiles than
8, counts around multiples of 8 and of the chip's blocks, cubes of one tile beside
cubes of hundreds, deep tiles beside shallow ones, and cubes that stop on the way
(the others' numbers move up). Every cube has the bits that it has alone; FP32 and
BF16 duals."""
import numpy as np
import pytest

from gpu_helpers import announce, dev, f32, torch_cuda
from synth.cubes import SMALL_64x64x16, like, make_cube
from test_gpu_step import STATE, get_state

pytestmark = pytest.mark.gpu

FEW = [(1, 8, 16), (2, 5, 7), (3, 8, 128)]
EIGHTS = [(n3, 8, 40 + n3) for n3 in range(1, 16)]
MIXED = [(40, 64, 128), (1, 3, 5), (9, 33, 131), (64, 17, 60), (2, 70, 90), (33, 8, 256), (7, 9, 11), (48, 40, 130)]


@pytest.mark.parametrize("dual", [0, 1])
@pytest.mark.parametrize("name,shapes,chunk", [("few", FEW, 1), ("eights", EIGHTS, 1), ("mixed", MIXED, 1),
                                               ("mixed", MIXED, 0)])
def test_batch_of_uneven_cubes(name, shapes, chunk, dual):
    announce(f"tiles of a batch: {name}, chunk {chunk}, dual storage {dual}")
    torch_cuda()
    import paper_2510_00562_amd as geo
    st = []
    for q, (n3, n1, n2) in enumerate(shapes):
        c = make_cube(like(SMALL_64x64x16, n1=n1, n2=n2, n3=n3, seed=70 + q, cells=5))
        # (every third cube stops by the rule after a few iterations)
        p = geo.params(max(c["eps"], 1e-3), c["alpha"], c["beta"], omega=0.03, dual_storage=dual, band_chunk=chunk,
                       max_iter=30, tol=0.2 if q % 3 == 1 else 0.0)
        d = geo.dims_of((n3, n1, n2))
        ws = geo.Workspace(geo.geo_workspace_size(d, p))
        vd = dev(f32(c["v"]))
        geo.geo_state_init(d, p, vd, ws)
        st.append((d, p, vd, ws))
    table = geo.Workspace(geo.geo_batch_table_size(len(st)))
    _, res = geo.geo_batch_step([x[0] for x in st], [x[1] for x in st], [x[2] for x in st], [x[3] for x in st], table,
                                20, use_graph=False)
    for shape, (d, p, vd, ws), r in zip(shapes, st, res):
        batch = get_state(geo, d, p, ws, vd, shape)
        geo.geo_state_init(d, p, vd, ws)
        solo = geo.geo_step(d, p, vd, ws, 20)
        assert (solo.iters, solo.tau_s, solo.tau_t, solo.r) == (r.iters, r.tau_s, r.tau_t, r.r), shape
        alone = get_state(geo, d, p, ws, vd, shape)
        for key in STATE:
            assert np.array_equal(alone[key], batch[key]), (shape, key)
    if name == "mixed":
        assert min(r.iters for r in res) < 20 and max(r.iters for r in res) == 20
