"""The search of the next thresholds at the end of an iteration (FP32 duals):
what it leaves for the next sweep has to survive the end of a call, and every
edge of the sweep's tiles (rows and columns around 8 x 128 and 16 x 64 tiles,
band chunks of one band left over, single rows, columns and bands).

25 iterations in one call, in 25 calls, and in calls of 1, 7 and 17 give the
same bits; the iterates follow the FP64 oracle. FP32 iterates round each of
about 30 operations per iteration at 6e-8: 25 iterations stay below 1e-5."""
import numpy as np
import pytest

from gpu_helpers import announce, dev, f32, rel_l2, torch_cuda
from synth.cubes import SMALL_64x64x16, like, make_cube
from test_gpu_step import STATE, get_state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(17, 9, 129), (9, 7, 127), (33, 16, 128), (8, 17, 65), (10, 15, 63),
                                   (1, 33, 64), (25, 1, 130), (9, 40, 1), (3, 24, 257)])
def test_iterations_split_over_calls(ora, shape):
    announce(f"25 iterations in one call and in several, {shape}")
    torch_cuda()
    import paper_2510_00562_amd as geo
    n3, n1, n2 = shape
    c = make_cube(like(SMALL_64x64x16, n1=n1, n2=n2, n3=n3, seed=31, cells=5))
    v = f32(c["v"])
    dims, vd = geo.dims_of(shape), dev(v)
    p = geo.params(c["eps"], c["alpha"], c["beta"], omega=0.03)
    runs = []
    for calls in ((25,), (1,) * 25, (1, 7, 17)):
        ws = geo.Workspace(geo.geo_workspace_size(dims, p))
        geo.geo_state_init(dims, p, vd, ws)
        for n in calls:
            r = geo.geo_step(dims, p, vd, ws, n)
            assert r.iters == n and r.slots == n
        runs.append((get_state(geo, dims, p, ws, vd, shape), (r.tau_s, r.tau_t, r.r, r.rel_change)))
    for s, sc in runs[1:]:
        assert sc == runs[0][1]
        for name in STATE:
            assert np.array_equal(s[name], runs[0][0][name]), name
    S = ora.Solver(v, c["eps"], c["alpha"], c["beta"], omega=0.03)
    S.step(25)
    for name in ("u", "s", "t"):
        assert rel_l2(runs[0][0][name], S.state[name]) <= 1e-5, name
