"""Pointwise projections of more values than one launch takes (2^35: 2^32 threads of
eight values each), in place in one buffer of 128 GiB: the box projection, and the
soft threshold that ends the l1 projection. Few distinct values, so every result is
known; values on either side of each launch's ends differ from their neighbours."""
import pytest

from gpu_helpers import announce, torch_cuda

pytestmark = pytest.mark.gpu

N = (1 << 35) + 5
MARKS = (0, 1 << 34, (1 << 34) - 1, (1 << 35) - 1, 1 << 35, N - 1)


@pytest.fixture(autouse=True)
def give_back():
    yield
    torch_cuda().cuda.empty_cache()


def buffer(torch):
    torch.cuda.empty_cache()
    free, _ = torch.cuda.mem_get_info()
    if free < 4 * N + (8 << 30):
        pytest.skip("needs 136 GiB of device memory")
    return torch.empty(N, dtype=torch.float32, device="cuda")


def check(torch, x, rest, mark):
    assert all(float(x[i]) == mark for i in MARKS)
    for q in range(0, N, 1 << 31):
        y = x[q:q + (1 << 31)]
        assert int((y != rest).sum()) == sum(q <= i < q + y.numel() for i in MARKS), q


def test_box():
    torch = torch_cuda()
    import paper_2510_00562_amd as geo
    announce(f"box projection of {N} values")
    x = buffer(torch).fill_(2.0)
    x[list(MARKS)] = 0.25
    geo.geo_project_box(x, 0.0, 1.0, x)
    check(torch, x, 1.0, 0.25)


def test_l1():
    torch = torch_cuda()
    import paper_2510_00562_amd as geo
    announce(f"l1 projection of {N} values")
    # |x| = 0.25, and 2 at the marks: tau = 1 with a radius of one above it each
    x = buffer(torch).fill_(-0.25)
    x[list(MARKS)] = 2.0
    tau = geo.geo_project_l1(x, float(len(MARKS)), x)
    assert tau == 1.0
    check(torch, x, 0.0, 1.0)
