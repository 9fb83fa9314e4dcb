"""Cubes of fewer voxels than the search of the next thresholds wants in a
window: the window must not grow past what the search's sums resolve. Every
threshold of 40 iterations against the FP64 oracle: within 1e-5 of it, or (where
it is small beside the values it cuts, up to about 1 and rounded at 6e-8 a few
times an iteration) 4e-7."""
import numpy as np
import pytest

from gpu_helpers import announce, dev, f32, torch_cuda
from synth.cubes import SMALL_64x64x16, like, make_cube

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("regularizer", [0, 1, 3])
@pytest.mark.parametrize("shape", [(3, 140, 1), (3, 140, 2), (5, 23, 31), (9, 9, 9), (2, 60, 70), (1, 50, 40)])
def test_thresholds_of_small_cubes(ora, shape, regularizer):
    announce(f"thresholds of a small cube {shape}, regularizer {regularizer}")
    torch_cuda()
    import paper_2510_00562_amd as geo
    n3, n1, n2 = shape
    c = make_cube(like(SMALL_64x64x16, n1=n1, n2=n2, n3=n3, seed=41, cells=5))
    v = f32(c["v"])
    dims, vd = geo.dims_of(shape), dev(v)
    p = geo.params(c["eps"], c["alpha"], c["beta"], omega=0.03, regularizer=regularizer)
    ws = geo.Workspace(geo.geo_workspace_size(dims, p))
    geo.geo_state_init(dims, p, vd, ws)
    if regularizer:
        S = ora.VariantSolver(v, c["eps"], c["alpha"], c["beta"], regularizer, omega=0.03)
    else:
        S = ora.Solver(v, c["eps"], c["alpha"], c["beta"], omega=0.03)
    for k in range(40):
        r = geo.geo_step(dims, p, vd, ws, 1)
        S.step(1)
        for got, want in zip((r.tau_s, r.tau_t), S.trace[-1][2:4]):
            assert got == pytest.approx(want, rel=1e-5, abs=4e-7), k
