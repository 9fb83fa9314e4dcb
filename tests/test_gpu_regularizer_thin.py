"""The comparison regularizers on cubes that 8 x 64 tiles fit badly: tiles fitted to
narrow cubes (idle threads, remainders of rows, one to 64 columns), one thread per
voxel where no tile is filled to 3/10 (spectra, single rows and columns, runs of
voxels that end within a band), and shapes on either side of the lines between the
three. Reference and tolerance as in test_gpu_regularizer_sweep.py. And the time of
an iteration over single spectra beside that of the same voxels in larger bands."""
import time

import numpy as np
import pytest

from gpu_helpers import announce, torch_cuda
from test_gpu_regularizer_sweep import check

pytestmark = pytest.mark.gpu

FITTED = [(9, 16, 16), (7, 70, 8), (3, 140, 4), (6, 71, 5), (33, 23, 21), (5, 25, 24), (2, 512, 30), (40, 20, 20),
          (3, 65, 33), (2, 2049, 6)]
FLAT = [(300, 1, 1), (70, 2, 3), (5, 70, 1), (40, 1, 66), (9, 8, 8), (3, 300, 2), (1, 5000, 1), (2, 2, 2048),
        (600, 50, 2), (3, 1, 1), (1, 1, 1)]
LINES = [(4, 153, 1), (4, 11, 14), (4, 11, 13), (4, 120, 70), (4, 112, 75)]


@pytest.mark.parametrize("variant", [1, 2, 3])
@pytest.mark.parametrize("shape", FITTED + FLAT + LINES)
def test_thin_cubes(variant, shape):
    announce(f"regularizer {variant}, thin cube {shape}")
    check(variant, shape)


def test_single_spectra_cost_no_multiple():
    """100000 voxels in one spectrum take less than three times an iteration of
    them in bands of 2500 (in 8 x 64 tiles fourteen times)."""
    torch = torch_cuda()
    import paper_2510_00562_amd as geo

    def us(shape):
        announce(f"SSTV on {shape}, timed")
        N = int(np.prod(shape))
        g = torch.Generator(device="cuda").manual_seed(1)
        v = 0.5 + 0.15 * torch.randn(shape, generator=g, device="cuda")
        p = geo.params(0.1 * np.sqrt(N), 0.004 * N, 0.002 * N, regularizer=1)
        d = geo.dims_of(shape)
        ws = geo.Workspace(geo.geo_workspace_size(d, p))
        geo.geo_state_init(d, p, v, ws)
        geo.geo_step(d, p, v, ws, 40)
        best = 1e9
        for _ in range(6):
            torch.cuda.synchronize()
            a = time.perf_counter()
            geo.geo_step(d, p, v, ws, 20)
            best = min(best, (time.perf_counter() - a) / 20 * 1e6)
        return best

    thin, wide = us((100000, 1, 1)), us((40, 50, 50))
    print(f"one spectrum {thin:.1f} us, 50 x 50 x 40 {wide:.1f} us", flush=True)
    assert thin <= 3.0 * wide
