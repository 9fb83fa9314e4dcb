"""The operators' two kernels against each other, on either side of 2^26 pixels a
band: a cube of two bands of 8192 x 8192 (the general kernel: one thread per output
element) against cubes of its rows that stay below (one thread per voxel), row by row
where an operator's outputs do not see the cut. And infinite inputs in bands large
enough for the kernel of one thread per voxel, which have to reach exactly the
outputs that the definition couples them to."""
import numpy as np
import pytest

from gpu_helpers import announce, torch_cuda
from test_gpu_ops_paths import OPS, run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("adjoint", [False, True])
@pytest.mark.parametrize("op", OPS)
def test_either_side_of_the_largest_band(op, adjoint):
    torch = torch_cuda()
    import paper_2510_00562_amd as geo
    n = 8192
    assert n * n == 1 << 26
    pin, pout = geo.OP_PLANES[op][:: -1 if adjoint else 1]
    announce(f"op {op} adjoint {adjoint}, bands of {n} x {n} pixels")
    g = torch.Generator(device="cuda").manual_seed(8)
    x = torch.randn((pin, 2, n, n), generator=g, device="cuda")

    def apply(rows):
        xs = x[:, :, rows].contiguous()
        out = torch.full((pout,) + xs.shape[1:], float("nan"), device="cuda")
        geo.geo_apply_op(op, adjoint, geo.dims_of(xs.shape[1:]), xs, out)
        return out

    whole = apply(slice(0, n))
    # at most 9 additions of FP32 terms, each within 6e-8 of the largest result
    tol = 9 * 6e-8 * float(whole.abs().max())
    top = apply(slice(0, n - 1))  # all but its last two rows see nothing of the cut
    assert float((whole[:, :, : n - 3] - top[:, :, : n - 3]).abs().max()) <= tol
    del top
    tail = apply(slice(n - 64, n))
    assert float((whole[:, :, n - 62:] - tail[:, :, 2:]).abs().max()) <= tol


@pytest.mark.parametrize("op,adjoint", [(op, adj) for op in ("dv", "dh", "ds", "d", "dds") for adj in (False, True)])
def test_infinite_values_in_bands_of_many_pixels(op, adjoint):
    torch = torch_cuda()
    import paper_2510_00562_amd as geo
    shape = (3, 15, 17)
    announce(f"op {op} adjoint {adjoint}: an infinite value, {shape}")
    pin = geo.OP_PLANES[op][1 if adjoint else 0]
    N = int(np.prod(shape))
    for at in (0, N - 1, 4 * 17 + 3, 16, pin * N - 1, pin * N - 17):
        x = np.zeros(pin * N)
        x[at] = 1.0
        touched = run(geo, torch, op, adjoint, shape, x) != 0
        x[at] = np.inf
        y = run(geo, torch, op, adjoint, shape, x)
        assert np.array_equal(~np.isfinite(y), touched), (at, np.flatnonzero(~np.isfinite(y) != touched))
