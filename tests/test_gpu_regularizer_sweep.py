"""The comparison regularizers' sweep at the sizes where its split can go wrong:
8 x 64 tiles with remainders of one row or column, band chunks with one band
left over, single rows, columns and bands, bands of more tiles than the search
has slots (4096: several tiles per slot), and bands of 2^27 pixels and more
(64-bit addresses instead of the buffer path).

The reference is the same iteration (eq. (7) with the step sizes of eq. (8)) in
64 bits. An iteration rounds each of about 10 operations on values of at most
about 2 at 6e-8 and its step sizes keep the iterates from growing: 5 iterations
stay below 5 * 10 * 1.2e-7 = 6e-6 in every element."""
import numpy as np
import pytest

from gpu_helpers import announce, torch_cuda

pytestmark = pytest.mark.gpu

ITERS = 5


def _threshold(torch, z, radius):
    """tau >= 0 with sum max(|z| - tau, 0) = radius (0 inside the ball)."""
    a = z.abs().reshape(-1)
    if float(a.sum()) <= radius:
        return 0.0
    a = a.sort(descending=True).values
    cs = a.cumsum(0)
    k = torch.arange(1, a.numel() + 1, device=a.device, dtype=torch.float64)
    keep = a * k > cs - radius
    n = int(keep.sum())
    return (float(cs[n - 1]) - radius) / n


def reference(torch, v, eps, alpha, beta, omega, variant, iters):
    def diff(x, dim):  # forward difference, 0 at the end
        y = torch.zeros_like(x)
        n = x.shape[dim]
        y.narrow(dim, 0, n - 1).copy_(x.narrow(dim, 1, n - 1) - x.narrow(dim, 0, n - 1))
        return y

    def diff_t(y, dim):
        x = torch.zeros_like(y)
        n = y.shape[dim]
        x.narrow(dim, 0, n - 1).sub_(y.narrow(dim, 0, n - 1))
        x.narrow(dim, 1, n - 1).add_(y.narrow(dim, 0, n - 1))
        return x

    v = v.double()
    na2 = 32.0 + (0.0 if variant == 1 else 8.0 * omega ** 2)
    gu, gt, gy = 1.0 / (na2 + 1.0), 0.2, 1.0 / 3.0
    u, s, t = v.clone(), torch.zeros_like(v), torch.zeros_like(v)
    y = [torch.zeros_like(v) for _ in range(2 if variant == 1 else 4)]
    y3, y4 = torch.zeros_like(v), torch.zeros_like(v)
    for _ in range(iters):
        g = diff_t(diff_t(y[0], 1) + diff_t(y[1], 2), 0)
        if variant > 1:
            g += omega * (diff_t(y[2], 1) + diff_t(y[3], 2))
        un = (u - gu * (g + y4)).clamp(0.0, 1.0)
        zs, zt = s - y4, t - gt * (diff_t(y3, 1) + y4)
        sn = zs.sign() * (zs.abs() - _threshold(torch, zs, alpha)).clamp_min(0.0)
        tn = zt.sign() * (zt.abs() - _threshold(torch, zt, beta)).clamp_min(0.0)
        up, sp, tp = 2.0 * un - u, 2.0 * sn - s, 2.0 * tn - t
        ds = diff(up, 0)
        ax = [diff(ds, 1), diff(ds, 2)]
        if variant > 1:
            ax += [omega * diff(up, 1), omega * diff(up, 2)]
        y = [a + gy * b for a, b in zip(y, ax)]
        if variant == 3:
            n = torch.sqrt(sum(a * a for a in y)).clamp_min(1.0)
            y = [a / n for a in y]
        else:
            y = [a.clamp(-1.0, 1.0) for a in y]
        y3 = y3 + gy * diff(tp, 1)
        q = y4 / gy + up + sp + tp - v
        y4 = gy * max(0.0, 1.0 - eps / float(q.norm())) * q
        u, s, t = un, sn, tn
    return dict(u=u, s=s, t=t, y1=torch.stack(y), y3=y3, y4=y4)


# (N3, N1, N2); (2, 2049, 1040) has 257 * 17 = 4369 tiles a band
@pytest.mark.parametrize("variant", [1, 2, 3])
@pytest.mark.parametrize("shape", [(9, 9, 65), (33, 8, 64), (17, 7, 63), (2, 16, 129), (1, 17, 128), (40, 1, 66),
                                   (12, 25, 1), (3, 8, 193), (2, 2049, 1040)])
def test_sweep_edges(variant, shape):
    announce(f"regularizer {variant}, sweep edges {shape}")
    check(variant, shape)


def test_bands_beyond_the_buffer_path():
    announce("a band of 16384 x 8193 pixels, 64-bit addresses")
    check(3, (1, 16384, 8193), scale=0.02)


def check(variant, shape, scale=1.0):
    torch = torch_cuda()
    import paper_2510_00562_amd as geo
    g = torch.Generator(device="cuda").manual_seed(5)
    N = int(np.prod(shape))
    v = 0.5 + 0.15 * torch.randn(shape, generator=g, device="cuda")
    # both l1 balls and the l2 ball active from the second iteration on
    eps, alpha, beta, omega = 0.02 * scale * np.sqrt(N), 0.004 * scale * N, 0.002 * scale * N, 0.07
    p = geo.params(eps, alpha, beta, omega=omega, regularizer=variant)
    dims = geo.dims_of(shape)
    ws = geo.Workspace(geo.geo_workspace_size(dims, p))
    geo.geo_state_init(dims, p, v, ws)
    geo.geo_step(dims, p, v, ws, 2)
    geo.geo_step(dims, p, v, ws, ITERS - 2)
    ref = reference(torch, v, eps, alpha, beta, omega, variant, ITERS)
    if scale < 1.0:
        # (one band moves only by the first-order term: smaller balls)
        assert all(float(ref[name].abs().max()) > 1e-4 for name in ref)
    for name, want in ref.items():
        got = torch.empty(want.shape, dtype=torch.float32, device="cuda")
        geo.geo_state_get(dims, p, ws, name, v, got)
        e = float((got.double() - want).abs().max())
        print(f"regularizer {variant} {shape} {name}: {e:.1e}", flush=True)
        assert e <= 6e-6, (name, e)


@pytest.mark.parametrize("seed", [4, 11])
def test_thresholds_of_late_iterations(seed):
    """Late in a solve the windows narrow with the steps of the thresholds: they
    hold, and the thresholds are those of the values (evaluated here in 64 bits from the FP32 state: 4
    roundings of 6e-8, and tau lies among the values that have them)."""
    announce(f"SSTV, late iterations, seed {seed}")
    torch = torch_cuda()
    import paper_2510_00562_amd as geo
    from gpu_helpers import dev, f32
    from synth.cubes import SMALL_64x64x16, like, make_cube
    shape = (198, 120, 120)
    c = make_cube(like(SMALL_64x64x16, n1=120, n2=120, n3=198, seed=seed, cells=20))
    v = dev(f32(c["v"]))
    dims = geo.dims_of(shape)
    p = geo.params(c["eps"], c["alpha"], c["beta"], regularizer=1)
    ws = geo.Workspace(geo.geo_workspace_size(dims, p))
    geo.geo_state_init(dims, p, v, ws)
    geo.geo_step(dims, p, v, ws, 900)
    for _ in range(3):
        assert geo.geo_step(dims, p, v, ws, 99).fallback_passes == 0
        x = {}
        for name in ("s", "t", "y3", "y4"):
            x[name] = torch.empty(shape, dtype=torch.float32, device="cuda")
            geo.geo_state_get(dims, p, ws, name, v, x[name])
        r = geo.geo_step(dims, p, v, ws, 1)
        x = {k: a.double() for k, a in x.items()}
        d = -x["y3"].clone()
        d[:, -1] = 0.0
        d[:, 1:] += x["y3"][:, :-1]
        want = (_threshold(torch, x["s"] - x["y4"], c["alpha"]),
                _threshold(torch, x["t"] - 0.2 * (d + x["y4"]), c["beta"]))
        print(f"tau {r.tau_s:.9g} {r.tau_t:.9g}, of the values {want[0]:.9g} {want[1]:.9g}; "
              f"in the windows {r.cand_s} {r.cand_t}", flush=True)
        assert r.tau_s == pytest.approx(want[0], rel=1e-6)
        assert r.tau_t == pytest.approx(want[1], rel=1e-6)
