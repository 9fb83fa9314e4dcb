"""The histogram passes of all missed thresholds in one launch: cubes so small
that one chunk of the voxels spans several of them, cubes whose two searches end
at different radix levels, a large cube beside them; every cube has the bits that
it has alone, where its chunks are others. FP32 and BF16 duals."""
import numpy as np
import pytest

from gpu_helpers import announce, dev, f32, torch_cuda
from synth.cubes import SMALL_64x64x16, like, make_cube
from test_gpu_step import STATE, get_state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dual", [0, 1])
def test_passes_over_many_small_cubes(dual):
    announce(f"histogram passes over 33 cubes, dual storage {dual}")
    torch_cuda()
    import paper_2510_00562_amd as geo
    shapes = [(1 + q % 3, 3 + q % 7, 5 + q % 11) for q in range(32)] + [(20, 70, 90)]
    st = []
    for q, (n3, n1, n2) in enumerate(shapes):
        c = make_cube(like(SMALL_64x64x16, n1=n1, n2=n2, n3=n3, seed=50 + q, cells=5))
        # (radii that the small cubes' values exceed from different iterations on)
        p = geo.params(max(c["eps"], 1e-3), 0.002 * n1 * n2 * n3 * (1 + q % 5), 0.001 * n1 * n2 * n3 * (1 + q % 3),
                       omega=0.03, dual_storage=dual, band_chunk=8)
        d = geo.dims_of((n3, n1, n2))
        ws = geo.Workspace(geo.geo_workspace_size(d, p))
        vd = dev(f32(c["v"]))
        geo.geo_state_init(d, p, vd, ws)
        st.append((d, p, vd, ws))
    table = geo.Workspace(geo.geo_batch_table_size(len(st)))
    _, res = geo.geo_batch_step([x[0] for x in st], [x[1] for x in st], [x[2] for x in st], [x[3] for x in st], table,
                                30, use_graph=True)
    assert sum(r.fallback_passes > 0 for r in res) > len(st) // 2
    for shape, (d, p, vd, ws), r in zip(shapes, st, res):
        batch = get_state(geo, d, p, ws, vd, shape)
        geo.geo_state_init(d, p, vd, ws)
        for _ in range(3):
            solo = geo.geo_step(d, p, vd, ws, 10)
        assert (solo.tau_s, solo.tau_t, solo.r) == (r.tau_s, r.tau_t, r.r), shape
        alone = get_state(geo, d, p, ws, vd, shape)
        for name in STATE:
            assert np.array_equal(alone[name], batch[name]), (shape, name)
