"""The projections and proximity operators over the sizes and alignments where
their loads of four values, their blocks and the histogram's packed sums can go
wrong: lengths around multiples of 4, 2048, 4096 and 65536 (the most values of
a block), pointers 4, 8 and 12 bytes off 16-byte alignment, in place, and values
that all fall into one bin.

Exact: soft threshold and box evaluate one rounding each, so the outputs are
compared with torch's FP64 evaluation rounded once; the threshold with a sort in
64 bits (1e-12 relative: sums of at most 2^23 values)."""
import pytest

from gpu_helpers import announce, torch_cuda

pytestmark = pytest.mark.gpu

SIZES = [1, 3, 4, 5, 2047, 2049, 4095, 4097, 65535, 65537, 262145, 1048579, 16777217]


def values(torch, n, seed, off):
    g = torch.Generator(device="cuda").manual_seed(seed)
    buf = torch.zeros(n + 8, device="cuda")
    x = buf[off:off + n]
    x.copy_(0.3 * torch.randn(n, generator=g, device="cuda"))
    return x


def threshold(torch, x, radius):
    a = x.double().abs().sort(descending=True).values
    cs = a.cumsum(0)
    if float(cs[-1]) <= radius:
        return 0.0
    k = torch.arange(1, a.numel() + 1, device=x.device, dtype=torch.float64)
    n = int((a * k > cs - radius).sum())
    return (float(a[:n].sum()) - radius) / n


@pytest.mark.parametrize("off", [0, 1, 2, 3])
@pytest.mark.parametrize("n", SIZES)
def test_l1_sizes(n, off):
    announce(f"l1 projection, n {n}, {4 * off} bytes off alignment")
    torch = torch_cuda()
    import paper_2510_00562_amd as geo
    x = values(torch, n, n, off)
    radius = 0.3 * float(x.double().abs().sum())
    want = threshold(torch, x, radius)
    m = x.double().abs() - want
    y = torch.where(m > 0, m.float().copysign(x), torch.zeros_like(x))
    out = torch.empty(n + 8, device="cuda")[(off + 1) % 4:][:n]
    tau = geo.geo_project_l1(x, radius, out)
    assert tau == pytest.approx(want, rel=1e-12)
    # (a threshold 1e-12 off moves a value by one rounding of itself at most)
    assert float((out - y).abs().max()) <= 6e-8 * float(x.abs().max())
    assert geo.geo_project_l1(x, radius, x) == tau  # in place
    assert torch.equal(x, out)


@pytest.mark.parametrize("n", [65536, 300000])
def test_l1_values_of_one_bin(n):
    announce(f"l1 projection, {n} equal values")
    torch = torch_cuda()
    import paper_2510_00562_amd as geo
    x = torch.full((n,), 1.9999999, device="cuda")
    out = torch.empty_like(x)
    radius = 0.25 * n
    tau = geo.geo_project_l1(x, radius, out)
    assert tau == pytest.approx(float(x[0].double()) - 0.25, rel=1e-14)


@pytest.mark.parametrize("off", [0, 1, 2, 3])
@pytest.mark.parametrize("n", SIZES)
def test_pointwise_sizes(n, off):
    announce(f"l2, l12, box, n {n}, {4 * off} bytes off alignment")
    torch = torch_cuda()
    import paper_2510_00562_amd as geo
    x, c = values(torch, n, n, off), values(torch, n, n + 1, (off + 2) % 4)
    out = torch.full((n + 8,), 7.0, device="cuda")
    o = out[(off + 1) % 4:][:n]
    geo.geo_project_box(x, -0.1, 0.2, o)
    assert torch.equal(o, x.clamp(-0.1, 0.2))
    e = (x.double() - c.double())
    norm = float(e.norm())
    r = geo.geo_project_l2(x, c, 0.5 * norm, o)
    assert r == pytest.approx(norm, rel=1e-12)
    assert float((o.double() - (c.double() + (0.5 * norm / r) * e)).abs().max()) <= 6e-8 * float(x.abs().max() + c.abs().max())
    assert geo.geo_project_l2(x, c, 2.0 * norm, o) == r and torch.equal(o, x)
    # the words around the output keep their values
    k = (off + 1) % 4
    assert bool((out[:k] == 7.0).all()) and bool((out[k + n:] == 7.0).all())
    oa, ob = torch.empty_like(x), torch.empty_like(x)
    geo.geo_prox_l12(x, c, 0.2, oa, ob)
    a, b = x.double(), c.double()
    f = (1.0 - 0.2 / (a * a + b * b).sqrt()).clamp_min(0.0)
    # the group's factor: 1 - 0.2 rsq, rounded a few times at 6e-8 of at most 1
    for got, want in ((oa, f * a), (ob, f * b)):
        assert float((got.double() - want).abs().max()) <= 5e-7 * float(x.abs().max() + c.abs().max())
