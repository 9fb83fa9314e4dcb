"""Operators on bands of few pixels, where one block per band and 256 pixels would
leave most lanes idle: every operator on both sides of the shares of lanes at which
the launch changes over (5/8, 3/8, 1/4 and 1/8 of 256), against the FP64 oracle, and the
time of one-pixel bands beside that of the same voxels in larger ones."""
import numpy as np
import pytest

from gpu_helpers import announce, f32, rel_l2, torch_cuda
from test_gpu_ops_paths import OPS, run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("adjoint", [False, True])
@pytest.mark.parametrize("op", OPS)
def test_both_sides_of_the_change(ora, op, adjoint):
    import paper_2510_00562_amd as geo
    torch = torch_cuda()
    for shape in [(300, 1, 1), (70, 2, 3), (9, 31, 1), (9, 4, 8), (9, 7, 9), (9, 8, 8), (5, 5, 19), (5, 16, 6),
                  (4, 53, 3), (4, 1, 160)]:
        announce(f"op {op} adjoint {adjoint} {shape}")
        pin = geo.OP_PLANES[op][1 if adjoint else 0]
        x = f32(np.random.default_rng(6).normal(size=pin * int(np.prod(shape))))
        xin = x if op == "k" else (x.reshape((pin,) + shape) if pin > 1 else x.reshape(shape))
        want = ora.apply(op, xin, shape, adjoint=adjoint).ravel()
        # at most 9 additions of FP32 terms, each within 6e-8 of the result's scale
        assert rel_l2(run(geo, torch, op, adjoint, shape, x), want) <= 1e-6


def test_bands_of_one_pixel_cost_no_multiple():
    """As many voxels in bands of one pixel and of 400: less than five times the
    time (a block for each pixel takes fourteen times)."""
    import paper_2510_00562_amd as geo
    torch = torch_cuda()

    def us(shape, adjoint):
        announce(f"K adjoint {adjoint} on {shape}, timed")
        pin, pout = geo.OP_PLANES["k"][:: -1 if adjoint else 1]
        x = torch.randn(pin * int(np.prod(shape)), device="cuda")
        out = torch.empty(pout * int(np.prod(shape)), device="cuda")
        e0, e1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        best = 1e9
        for _ in range(6):
            e0.record()
            for _ in range(20):
                geo.geo_apply_op("k", adjoint, geo.dims_of(shape), x, out)
            e1.record()
            torch.cuda.synchronize()
            best = min(best, e0.elapsed_time(e1) / 20 * 1e3)
        return best

    for adjoint in (False, True):
        thin, wide = us((100000, 1, 1), adjoint), us((250, 20, 20), adjoint)
        print(f"one pixel {thin:.1f} us, 400 pixels {wide:.1f} us", flush=True)
        assert thin <= 5.0 * wide
