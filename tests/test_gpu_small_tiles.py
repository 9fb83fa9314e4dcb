"""The sweep's small form (256 threads, cubes whose bands are one tile of at most 256
pixels, 40 rows and columns together and 32 columns; BF16 duals: 8 rows and more than
256 bands): its largest tiles, single pixels, rows and columns, and the first sizes
past each limit, with FP32 and BF16 duals; many chunks of bands, one band each and
bands left over; with cubes of the other forms in one batch, in a launch of its own
and among their tiles. Tolerances are those of the tests whose checks are used. And
the time of an iteration over single spectra beside that of as many voxels in larger
bands."""
import time

import numpy as np
import pytest

from gpu_helpers import announce, torch_cuda
from test_gpu_step import STATE, get_state
from test_gpu_step import test_one_step_from_random_state as one_step
from test_gpu_tiles import setup
from test_gpu_tiles import test_fitted_tiles_follow_the_oracle as follow_the_oracle
from test_gpu_workloads import test_bf16_duals_one_step as bf16_one_step

pytestmark = pytest.mark.gpu

# (N3, N1, N2)
SMALL = [(5, 16, 16), (3, 8, 32), (3, 32, 8), (4, 38, 2), (6, 1, 32), (9, 39, 1), (40, 1, 1), (7, 13, 19), (300, 3, 3)]
PAST = [(3, 1, 33), (3, 17, 16), (3, 36, 5), (3, 40, 1), (3, 9, 31)]


@pytest.mark.parametrize("shape", SMALL + PAST)
def test_one_step(ora, shape):
    one_step(ora, shape)


@pytest.mark.parametrize("shape", [(260, 8, 32), (257, 9, 16), (270, 1, 32), (400, 1, 1), (256, 8, 19), (300, 3, 3),
                                   (40, 8, 5)])
def test_one_step_bf16(ora, shape):
    bf16_one_step(ora, shape)


@pytest.mark.parametrize("shape,chunk", [((5000, 1, 1), 0), ((5000, 1, 1), 9), ((1100, 4, 5), 0), ((70, 16, 16), 0),
                                         ((70, 16, 16), 8)])
def test_many_chunks(ora, shape, chunk):
    follow_the_oracle(ora, shape, chunk)


@pytest.mark.parametrize("shapes", [
    # 743 small tiles: a launch of their own
    [(40, 9, 11), (5, 33, 33), (9, 24, 128), (700, 1, 2), (3, 16, 16), (12, 16, 256)],
    # 43 and 256: with the others, in 1024 threads (alone in 256)
    [(40, 9, 11), (5, 33, 33), (9, 24, 128), (3, 16, 16), (12, 16, 256)],
    [(250, 16, 16), (6, 7, 30), (9, 24, 128)],
])
def test_every_form_in_one_batch(shapes):
    """Small tiles, fitted ones and 8 x 128: the bits of each cube alone."""
    announce(f"small, fitted and fixed tiles in one batch: {shapes}")
    torch_cuda()
    import paper_2510_00562_amd as geo
    st = [setup(s, 0) for s in shapes]
    table = geo.Workspace(geo.geo_batch_table_size(len(st)))
    geo.geo_batch_step([x[2] for x in st], [x[4] for x in st], [x[3] for x in st], [x[5] for x in st], table, 20,
                       use_graph=True)
    for shape, (_, _, dims, vd, p, ws) in zip(shapes, st):
        batch = get_state(geo, dims, p, ws, vd, shape)
        geo.geo_state_init(dims, p, vd, ws)
        geo.geo_step(dims, p, vd, ws, 20)
        solo = get_state(geo, dims, p, ws, vd, shape)
        for name in STATE:
            assert np.array_equal(solo[name], batch[name]), (shape, name)


@pytest.mark.parametrize("dual,most", [(0, 30.0), (1, 12.0)])
def test_single_spectra(dual, most):
    """100000 voxels in one spectrum against as many in bands of 2500: 14 times an
    iteration with FP32 duals, 5.5 with BF16; in workgroups of 1024 threads 57 and
    22 times."""
    torch = torch_cuda()
    import paper_2510_00562_amd as geo

    def us(shape):
        announce(f"GeoSSTV on {shape}, dual storage {dual}, timed")
        N = int(np.prod(shape))
        g = torch.Generator(device="cuda").manual_seed(1)
        v = 0.5 + 0.15 * torch.randn(shape, generator=g, device="cuda")
        p = geo.params(0.1 * np.sqrt(N), 0.004 * N, 0.002 * N, dual_storage=dual)
        d = geo.dims_of(shape)
        ws = geo.Workspace(geo.geo_workspace_size(d, p))
        geo.geo_state_init(d, p, v, ws)
        geo.geo_step(d, p, v, ws, 40)
        best = 1e9
        for _ in range(4):
            torch.cuda.synchronize()
            a = time.perf_counter()
            geo.geo_step(d, p, v, ws, 20)
            best = min(best, (time.perf_counter() - a) / 20 * 1e6)
        return best

    thin, wide = us((100000, 1, 1)), us((40, 50, 50))
    print(f"one spectrum {thin:.1f} us, 50 x 50 x 40 {wide:.1f} us", flush=True)
    assert thin <= most * wide
