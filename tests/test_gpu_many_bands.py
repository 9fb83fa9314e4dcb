"""Operators on cubes of very many bands: as many blocks as bands are more than one
launch takes (2^32 threads), whether a band fills a block or holds one pixel.
Against torch's differences of the same floats, which round once: equal."""
import pytest

from gpu_helpers import announce, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1 << 24, 1, 1), ((1 << 24) + 3, 2, 1), ((1 << 23) + 5, 10, 16)])
def test_differences_over_many_bands(shape):
    announce(f"ds and dv on {shape}")
    torch = torch_cuda()
    import paper_2510_00562_amd as geo
    g = torch.Generator(device="cuda").manual_seed(3)
    x = torch.randn(shape, generator=g, device="cuda")
    out = torch.full(shape, float("nan"), device="cuda")
    dims = geo.dims_of(shape)
    for op, dim in (("ds", 0), ("dv", 1)):
        n = shape[dim] - 1
        geo.geo_apply_op(op, False, dims, x, out)
        assert not out.narrow(dim, n, 1).any()
        if n:
            assert torch.equal(out.narrow(dim, 0, n), x.narrow(dim, 1, n) - x.narrow(dim, 0, n)), op
        geo.geo_apply_op(op, True, dims, x, out)
        want = torch.zeros_like(x)
        if n:
            want.narrow(dim, 1, n).copy_(x.narrow(dim, 0, n))
            want.narrow(dim, 0, n).sub_(x.narrow(dim, 0, n))
        assert torch.equal(out, want), op
        out.fill_(float("nan"))
