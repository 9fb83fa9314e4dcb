"""Thresholds at the boundary of the l1 ball: sum |z| exceeds the radius by 2e-5 of
it, which is outside, in a cube of 4096 bands taken by one tile (a sum in 32 bits
over a tile's bands would be low by 3.4e-5 and take it for inside).

The state makes every value known: u constant, everything else zero. After one
iteration y4 = a4 q with q = u - v and a4 = 0.2 (eps = 0), so z_s = -y4 and
z_t = -step y4 are the same number everywhere and tau = |z| - radius / N. The values are FP32 and the
sums FP64: relative error below 1e-9 of |z|."""
import numpy as np
import pytest

from gpu_helpers import announce, torch_cuda

pytestmark = pytest.mark.gpu

SHAPE = (4096, 8, 8)
Q = np.float32(2542 / 8192)


@pytest.mark.parametrize("field", ["s", "t"])
def test_just_outside_the_ball(field):
    announce(f"sum |z_{field}| 2e-5 above the radius, 4096 bands in one tile")
    torch = torch_cuda()
    import paper_2510_00562_amd as geo
    z = np.float32(0.2) * Q
    if field == "t":  # z_t = fma(-step, y4, 0), step and y4 rounded to FP32
        z = np.float32(np.float64(np.float32(1.0 / 3.0)) * np.float64(z))
    s = np.add.accumulate(np.full(SHAPE[0], z, np.float32), dtype=np.float32)[-1]
    assert float(s) < SHAPE[0] * float(z) * (1 - 3.4e-5)  # the sum that 32 bits would give
    N = int(np.prod(SHAPE))
    radius = float(z) * N * (1 - 2e-5)
    alpha, beta = (radius, 1e9) if field == "s" else (1e9, radius)
    v = torch.full(SHAPE, 0.5, device="cuda")
    dims = geo.dims_of(SHAPE)
    p = geo.params(0.0, alpha, beta, omega=0.03, band_chunk=SHAPE[0])
    ws = geo.Workspace(geo.geo_workspace_size(dims, p))
    geo.geo_state_init(dims, p, v, ws)
    geo.geo_state_set(dims, p, ws, "u", v, v + float(Q))
    r = geo.geo_step(dims, p, v, ws, 2)
    tau = r.tau_s if field == "s" else r.tau_t
    print(f"tau {tau:.6e}, of the values {float(z) - radius / N:.6e}, r {r.r:.6e}", flush=True)
    assert abs(tau - (float(z) - radius / N)) <= 1e-9 * float(z)
